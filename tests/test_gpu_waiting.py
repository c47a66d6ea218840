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


@pytest.mark.parametrize("power", [300, -300])
def test_buckets_at_any_scale_of_time(gpu, oracle_lib, power):
    """Speeds, bucket width and start time scaled by a power of two: the keys
    that order the work keep the range of the times, so the buckets are walked
    as they are unscaled, and the times are the unscaled ones scaled."""
    f = np.random.default_rng(9).uniform(1.0, 3.0, (33, 70, 90))
    src = torch.tensor([0])
    kw = dict(tile=(8, 8, 8), lookahead=0, check_status=False)
    adv = []
    for p in (0, power):
        t = gpu.solve(torch.from_numpy(np.ldexp(f, -p)).cuda(), 1.0, src, delta=float(np.ldexp(0.5, p)), **kw)
        adv.append(gpu.status().bucket_advances)
        if p == 0:
            ref = t.cpu().numpy()
            assert np.array_equal(ref.view(np.uint64), oracle_lib.fmm(f, 1.0, src.numpy()).reshape(f.shape).view(np.uint64))
        else:
            assert np.array_equal(t.cpu().numpy().view(np.uint64), np.ldexp(ref, p).view(np.uint64))
    print(adv)
    assert adv[0] > 40 and adv[1] > adv[0] / 2


def test_strict_window_keeps_the_bucket_order(gpu):
    """With narrow buckets idle workers find work only above the window.  Kept
    from it they take the buckets one by one: more advances, fewer early runs,
    the same times and gradients."""
    import workloads as W
    p = W.layered_3d(160, 150, 100, h=10.0, seed=3)
    f, src = torch.from_numpy(p.field).cuda(), torch.as_tensor(p.src).cuda()
    g = torch.ones_like(f)
    runs, advances, times, grads = [], [], [], []
    for strict in (False, True):
        t, par = gpu.solve(f, p.h, src, parents=True, tile=(8, 8, 8), delta=0.002, lookahead=0, strict_window=strict)
        st = gpu.status()
        runs.append(st.tile_visits)
        advances.append(st.bucket_advances)
        times.append(t)
        grads.append(gpu.adjoint(f, p.h, t, par, g, tile=(8, 8, 8), delta=0.002, strict_window=strict))
    print(runs, advances)
    assert runs[1] < 0.85 * runs[0] and advances[1] > 1.2 * advances[0]
    assert torch.equal(times[0], times[1]) and torch.equal(grads[0], grads[1])
