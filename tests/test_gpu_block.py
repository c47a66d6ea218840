"""Launches of few tiles run on a workgroup per tile, all others on a wave per
tile.  Here each form is run on the other's ground (a bound on the workgroups
keeps a launch on the wave-per-tile kernels) and on both sides of the line
between them, against the oracle: times bitwise, gradients within 1e-12
relative (the same operations in the same order)."""
import numpy as np
import pytest
import torch

import workloads as W
from test_gpu_sweep import TILES, check

pytestmark = pytest.mark.gpu
WAVES = dict(grid_blocks=4096)  # more than fit: no bound, but the wave-per-tile kernels


@pytest.fixture(scope="module")
def O(oracle_lib):
    return oracle_lib


def edge_shapes(tile):
    tx, ty, tz = tile
    for d in (-1, 0, 1):
        yield (1 if tz == 1 else max(tz + d, 2), max(2 * ty - d, 2), max(tx + d, 2))


@pytest.mark.parametrize("tile", TILES)
def test_waves_on_small_grids(gpu, O, tile):
    rng = np.random.default_rng(300 + sum(tile))
    kt = dict(tile=tile if tile[2] > 1 else tile[:2], **WAVES)
    for shape in edge_shapes(tile):
        f = W.random_field(shape, rng, 0.5, 5.0, block=3)
        n = f.size
        src = np.unique(np.array([0, n - 1, rng.integers(0, n)], dtype=np.int64))
        for kw in (dict(), dict(delta=1.5, lookahead=3), dict(delta=2.0, horizon=1)):
            check(gpu, O, f, src, **kw, **kt)
            check(gpu, O, f, src[:1], **kw, **kt)
        # stopped by the visit cap, then resumed
        ref = O.fmm(f, 1.0, src).reshape(shape)
        fd, sd = torch.from_numpy(f if shape[0] > 1 else f[0]).cuda(), torch.from_numpy(src)
        t = gpu.solve(fd, 1.0, sd, max_tile_visits=2, check_status=False, **kt)
        gpu.status(raise_on_error=False)
        t = gpu.solve(fd, 1.0, sd, out=t, warm_start=True, **kt)
        assert np.array_equal(t.cpu().numpy().reshape(shape).view(np.uint64), ref.view(np.uint64)), shape
        ax = [np.cumsum(10.0 ** rng.uniform(-0.5, 0.5, m)) for m in shape[::-1]]
        rr = O.solve_rect(f, ax[0], ax[1], ax[2] if shape[0] > 1 else None, src).reshape(shape)
        got = gpu.solve_rect(fd, ax[0], ax[1], ax[2] if shape[0] > 1 else None, sd, **kt)
        assert np.array_equal(got.cpu().numpy().reshape(shape).view(np.uint64), rr.view(np.uint64)), shape


@pytest.mark.parametrize("tile", TILES)
def test_adjoint_waves_on_small_grids(gpu, O, tile):
    rng = np.random.default_rng(400 + sum(tile))
    for shape in edge_shapes(tile):
        f = W.random_field(shape, rng, 0.5, 5.0, block=2)
        src = np.unique(rng.integers(0, f.size, 3)).astype(np.int64)
        t = O.fmm(f, 1.0, src)
        par = O.parents(t, src)
        g = rng.standard_normal(shape)
        ref = O.adjoint(t, par, f, 1.0, g).reshape(shape)
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a.reshape(shape)[0 if shape[0] == 1 else slice(None)])).cuda()
        for kw in (dict(), dict(delta=1.0, lookahead=4)):
            got = gpu.adjoint(dev(f), 1.0, dev(t), dev(par), dev(g), tile=tile if tile[2] > 1 else tile[:2], **kw, **WAVES)
            err = np.max(np.abs(got.cpu().numpy().reshape(shape) - ref)) / np.max(np.abs(ref))
            assert err <= 1e-12, (shape, kw, err)


@pytest.mark.parametrize("tile,shape", [((16, 8, 8), (64, 64, 256)), ((16, 8, 8), (64, 64, 257)), ((8, 8, 8), (64, 128, 64)),
                                        ((8, 8, 8), (65, 128, 64)), ((32, 32, 1), (1, 32, 32)), ((32, 32, 1), (1, 32, 33))])
def test_solves_about_the_line(gpu, O, tile, shape):
    """1024 tiles of one problem and more in 3D, one tile and two in 2D."""
    rng = np.random.default_rng(sum(shape))
    f = W.random_field(shape, rng, 0.5, 3.0, block=4)
    src = rng.integers(0, f.size, 2).astype(np.int64)
    for kw in (dict(), dict(delta=3.0, lookahead=4)):
        check(gpu, O, f, src, tile=tile if tile[2] > 1 else tile[:2], **kw)


@pytest.mark.parametrize("tile,n", [((16, 8, 8), 800), ((16, 8, 8), 801), ((16, 8, 8), 1600), ((16, 8, 8), 1601),
                                    ((8, 8, 8), 400), ((32, 32), 24), ((32, 32), 25), ((32, 32), 101), ((32, 32), 226)])
def test_batches_about_the_line(gpu, O, tile, n):
    """800 and 1600 problems of one tile, 25 and more of four tiles in 2D, each with
    and without one more; forward, parents and adjoint."""
    rng = np.random.default_rng(n)
    shapes = [(5, 7, 9), (8, 8, 16), (3, 8, 11)] if len(tile) == 3 else [(1, 33, 40), (1, 64, 64), (1, 50, 34)]
    fields = [W.random_field(shapes[i % 3], rng, 0.5, 4.0) for i in range(n)]
    srcs = [np.array([rng.integers(0, f.size)], dtype=np.int64) for f in fields]
    b = gpu.pack([torch.from_numpy(f if f.shape[0] > 1 else f[0]).cuda() for f in fields], 1.0, [torch.from_numpy(s) for s in srcs])
    t = torch.empty(b.npts, dtype=torch.float64, device="cuda")
    par = torch.empty(b.npts, dtype=torch.uint8, device="cuda")
    g = torch.from_numpy(rng.standard_normal(b.npts)).cuda()
    grad = torch.empty_like(t)
    gpu.solve_packed(b, t, par, tile=tile)
    gpu.status()
    gpu.adjoint_packed(b, t, par, g, grad, tile=tile)
    gpu.status()
    ts, ps, gs, rs = b.views(t), b.views(par), b.views(g), b.views(grad)
    for i in range(0, n, 17):
        ref = O.fmm(fields[i], 1.0, srcs[i])
        assert np.array_equal(ts[i].cpu().numpy().ravel().view(np.uint64), ref.ravel().view(np.uint64)), i
        rp = O.parents(ref, srcs[i])
        assert np.array_equal(ps[i].cpu().numpy().ravel(), rp.ravel()), i
        ra = O.adjoint(ref, rp, fields[i], 1.0, gs[i].cpu().numpy()).ravel()
        assert np.max(np.abs(rs[i].cpu().numpy().ravel() - ra)) <= 1e-12 * np.max(np.abs(ra)), i


@pytest.mark.parametrize("shape", [(64, 80, 160), (65, 80, 160), (24, 24, 24)])
def test_adjoints_about_the_line(gpu, O, shape):
    """800 tiles of 16x8x8 and more."""
    rng = np.random.default_rng(sum(shape))
    for sh in (shape,):
        f = W.random_field(sh, rng, 0.5, 5.0, block=2)
        src = np.unique(rng.integers(0, f.size, 2)).astype(np.int64)
        t = O.fmm(f, 1.0, src)
        par = O.parents(t, src)
        g = rng.standard_normal(sh)
        ref = O.adjoint(t, par, f, 1.0, g).reshape(sh)
        d = lambda a: torch.from_numpy(np.ascontiguousarray(a.reshape(sh))).cuda()
        got = gpu.adjoint(d(f), 1.0, d(t), d(par), d(g)).cpu().numpy()
        assert np.max(np.abs(got - ref)) <= 1e-12 * np.max(np.abs(ref)), sh
