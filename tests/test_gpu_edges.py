"""Values and uses at the edge of the rewritten kernels: gradients and stored
times that are infinite or NaN, and solves on several streams and threads at
once.  Both forms of the kernels (a bound on the workgroups keeps a launch on
the wave-per-tile ones)."""
import threading

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu
FORMS = [dict(), dict(grid_blocks=4096)]


@pytest.mark.parametrize("shape,tile", [((1, 70, 45), (32, 32)), ((19, 21, 37), (16, 8, 8)), ((19, 21, 37), (8, 8, 8))])
def test_upstream_gradients_not_finite(gpu, oracle_lib, shape, tile):
    """A NaN reaches every point it flows to and no other; infinities behave as in
    the oracle, which does the same operations in the same order."""
    rng = np.random.default_rng(sum(shape))
    f = W.random_field(shape, rng, 0.5, 3.0, block=3)
    src = np.unique(rng.integers(0, f.size, 2)).astype(np.int64)
    t = oracle_lib.fmm(f, 1.0, src)
    par = oracle_lib.parents(t, src)
    sq = lambda a: np.ascontiguousarray(a.reshape(shape)[0] if shape[0] == 1 else a.reshape(shape))
    dev = lambda a: torch.from_numpy(sq(a)).cuda()
    for bad in (np.nan, np.inf, -np.inf, (np.inf, -np.inf), (np.nan, np.inf)):
        g = rng.standard_normal(f.size)
        vals = bad if isinstance(bad, tuple) else (bad,)
        for v in vals:
            g[rng.integers(0, f.size, 3)] = v
        with np.errstate(all="ignore"):
            ref = sq(oracle_lib.adjoint(t, par, f, 1.0, g.reshape(shape)))
        for kw in FORMS:
            got = gpu.adjoint(dev(f), 1.0, dev(t), dev(par), dev(g), tile=tile, **kw).cpu().numpy()
            assert np.array_equal(np.isnan(got), np.isnan(ref)), (bad, kw)
            inf = np.isinf(ref)
            assert np.array_equal(got[inf], ref[inf]), (bad, kw)
            ok = np.isfinite(ref)
            assert np.max(np.abs(got[ok] - ref[ok])) <= 1e-12 * np.max(np.abs(ref[ok])), (bad, kw)


def parents_by_hand(t):
    """The parent byte of every point of t [nz, ny, nx] as eik.h states it; a value
    with its sign bit set counts as a source."""
    a = np.abs(t)
    out = np.zeros(t.shape, dtype=np.uint8)
    for k, ax in enumerate((2, 1, 0)):
        pad = [(1, 1) if i == ax else (0, 0) for i in range(3)]
        p = np.pad(a, pad, constant_values=np.inf)
        lo = np.take(p, range(0, t.shape[ax]), ax)
        hi = np.take(p, range(2, t.shape[ax] + 2), ax)
        with np.errstate(invalid="ignore"):
            up = np.fmin(lo, hi) < t
            out |= np.where(up, np.where(lo <= hi, 1, 2), 0).astype(np.uint8) << (2 * k)
    return np.where(np.signbit(t), np.uint8(0x80), out)


@pytest.mark.parametrize("nx", [1, 3, 4, 7, 64, 129])
def test_parent_record_of_times_not_finite(gpu, nx):
    rng = np.random.default_rng(nx)
    t = rng.uniform(0.0, 2.0, (5, 9, nx))
    for v in (np.nan, np.inf, -0.0, 0.0, -1.0, 1.0):
        t[rng.random(t.shape) < 0.08] = v
    want = parents_by_hand(t)
    want[0, 0, 0] = 0x80
    got = gpu.parents_of(torch.from_numpy(t).cuda(), torch.tensor([0])).cpu().numpy()
    assert np.array_equal(got, want)


def test_streams_and_threads(gpu, oracle_lib):
    """Four threads, a stream each, solves and adjoints of their own sizes at
    once, status read each time: every result is that of the problem alone."""
    rng = np.random.default_rng(12)
    jobs = []
    for i, shape in enumerate(((33, 40, 50), (90, 100, 110), (12, 9, 20), (64, 64, 64))):
        f = W.random_field(shape, rng, 0.5, 4.0, block=4)
        src = rng.integers(0, f.size, 2).astype(np.int64)
        ref = oracle_lib.fmm(f, 1.0, src).reshape(shape)
        jobs.append((torch.from_numpy(f).cuda(), torch.from_numpy(src).cuda(), torch.from_numpy(ref).cuda(),
                     torch.from_numpy(rng.standard_normal(shape)).cuda(), FORMS[i % 2], torch.cuda.Stream()))
    alone = []
    for f, src, ref, g, kw, _ in jobs:
        t, par = gpu.solve(f, 1.0, src, parents=True, delta=1.0, lookahead=4, **kw)
        alone.append((par.clone(), gpu.adjoint(f, 1.0, t, par, g, **kw).clone()))
    torch.cuda.synchronize()
    errors = []

    def work(job, want):
        f, src, ref, g, kw, stream = job
        try:
            with torch.cuda.stream(stream):
                for _ in range(12):
                    t, par = gpu.solve(f, 1.0, src, parents=True, delta=1.0, lookahead=4, **kw)
                    grad = gpu.adjoint(f, 1.0, t, par, g, **kw)
                    stream.synchronize()
                    if not (torch.equal(t, ref) and torch.equal(par, want[0]) and torch.equal(grad, want[1])):
                        errors.append(tuple(f.shape))
        except Exception as e:  # noqa: BLE001 -- reported below, in the main thread
            errors.append(repr(e))

    threads = [threading.Thread(target=work, args=(j, w)) for j, w in zip(jobs, alone)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert not errors, errors
