"""A worker that waits tells a launch that makes progress from one that does not."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_channel_longer_than_the_watchdog(gpu, oracle_lib):
    """A front along one row is handed on from tile to tile: the rings' counts
    stand still for the whole solve, here (about 18 s) longer than the 14 s that
    a launch without progress is given.  With few workgroups the polls are the
    most frequent."""
    n = 24_000_000
    f = np.random.default_rng(3).uniform(1.0, 2.0, (1, 1, n))
    src = np.array([0], dtype=np.int64)
    t = gpu.solve(torch.from_numpy(f[0]).cuda(), 1.0, torch.from_numpy(src), tile=(16, 8), grid_blocks=4,
                  time_kernels=True, check_status=False)
    st = gpu.status()
    print(f"{st.kernel_ms:.0f} ms, {st.handoffs} hand-ons of {st.tile_visits} runs")
    assert st.handoffs > 0.9 * st.tile_visits
    ref = oracle_lib.fmm(f, 1.0, src)
    assert np.array_equal(t.cpu().numpy().ravel().view(np.uint64), ref.ravel().view(np.uint64))
