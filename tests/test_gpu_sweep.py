"""The wave-per-tile solver and adjoint and the sharded bucket rings at the sizes where they
can go wrong: grids one point short of, at and one past a tile's edges, grids
thinner than a tile, single tiles, a few tiles (fewer than the shards, not a
multiple of 8), fronts from every octant and from several sides at once,
sources on tile corners, and batches of more problems than a wave has lanes.
Every time is bitwise the oracle's; gradients are within 1e-12 relative of the
oracle's (the same operations in the same order)."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

TILES = [(32, 8, 4), (16, 8, 8), (8, 8, 8), (64, 4, 4), (16, 8, 4), (8, 8, 4), (8, 4, 4),
         (32, 32, 1), (64, 16, 1), (128, 8, 1), (16, 16, 1), (16, 8, 1)]


@pytest.fixture(scope="module")
def O(oracle_lib):
    return oracle_lib


def check(eik, O, field, src, t0=None, **kw):
    ref = O.fmm(field, 1.0, src, t0=t0)
    f = torch.from_numpy(field if field.shape[0] > 1 else field[0]).cuda()
    got = eik.solve(f, 1.0, torch.from_numpy(src), t0=None if t0 is None else torch.from_numpy(t0), **kw)
    got = got.cpu().numpy().reshape(field.shape)
    assert np.array_equal(got.view(np.uint64), ref.reshape(field.shape).view(np.uint64)), (field.shape, kw)


@pytest.mark.parametrize("tile", TILES)
def test_tile_edges(gpu, O, tile):
    rng = np.random.default_rng(sum(tile))
    tx, ty, tz = tile
    for d in (-1, 0, 1):
        for e in (-1, 1):
            nz = 1 if tz == 1 else max(tz + d, 2)
            shape = (nz, max(2 * ty + e, 2), max(tx + d, 2))
            f = W.random_field(shape, rng, 0.5, 5.0, block=3)
            n = f.size
            # the corners of the grid and of the tiles, all octants at once
            src = np.unique(np.array([0, n - 1, shape[2] - 1, min(tx, shape[2]) - 1, rng.integers(0, n)],
                                     dtype=np.int64))
            for s in (src, src[-1:], src[:1]):
                check(gpu, O, f, s, tile=tile if tz > 1 else tile[:2], delta=1.5, lookahead=3)


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 1, 300), (1, 300, 1), (2, 2, 2), (3, 1, 200), (200, 3, 1), (9, 65, 17),
                                   (17, 9, 130)])
def test_thin_and_few_tiles(gpu, O, shape):
    rng = np.random.default_rng(sum(shape))
    f = W.random_field(shape, rng, 0.2, 3.0)
    src = np.array([rng.integers(0, f.size)], dtype=np.int64)
    tiles = [(16, 8, 8), (8, 4, 4)] if shape[0] > 1 else [(32, 32), (16, 8)]
    for tile in tiles:
        for kw in (dict(), dict(delta=0.7, lookahead=16), dict(delta=2.0, horizon=1)):
            check(gpu, O, f, src, np.array([0.25]), tile=tile, **kw)


def test_batch_beyond_a_wave(gpu, O):
    """130 problems: the wave finds a tile's problem in steps of 64."""
    rng = np.random.default_rng(8)
    fields, srcs = [], []
    for i in range(130):
        f = W.random_field(tuple(int(v) for v in rng.integers(3, 19, 3)), rng, 0.5, 4.0)
        fields.append(f)
        srcs.append(np.array([rng.integers(0, f.size)], dtype=np.int64))
    ts = gpu.solve_batched([torch.from_numpy(f).cuda() for f in fields], 1.0, [torch.from_numpy(s) for s in srcs],
                           delta=0.5, tile=(8, 8, 8), lookahead=8)
    for f, s, t in zip(fields, srcs, ts):
        ref = O.fmm(f, 1.0, s)
        assert np.array_equal(t.cpu().numpy().view(np.uint64), ref.reshape(f.shape).view(np.uint64)), f.shape


def test_values_that_miss_the_window(gpu, O):
    """Constants far below an ulp of the times, and equal minima: the short form
    of the operator must hand these to the exact search."""
    rng = np.random.default_rng(4)
    f = W.random_field((9, 17, 19), rng, 1.0, 2.0)
    f[:, 4:12, 5:14] *= 1e13
    src = np.array([0, f.size // 2], dtype=np.int64)
    check(gpu, O, f, src, np.array([1000.0, 1000.0]), tile=(8, 8, 8), delta=0.5, lookahead=4)
    g = np.full((1, 40, 40), 3.0)
    check(gpu, O, g, np.array([0, 39, 1599], dtype=np.int64), tile=(16, 16), delta=1.0)


@pytest.mark.parametrize("tile", TILES)
def test_rectilinear_tile_edges(gpu, O, tile):
    """Spacings over six decades: axes that drop out of the root, equal minima
    with different weights on the two sides, and values that miss the window of
    three doubles."""
    rng = np.random.default_rng(200 + sum(tile))
    tx, ty, tz = tile
    axis = lambda n, lo, hi: np.cumsum(10.0 ** rng.uniform(lo, hi, n))
    for d, lo, hi in ((-1, -0.5, 0.5), (0, -3.0, 3.0), (1, -0.1, 0.1)):
        nz = 1 if tz == 1 else max(tz + d, 2)
        shape = (nz, max(2 * ty - d, 2), max(tx + d, 2))
        f = W.random_field(shape, rng, 0.5, 5.0, block=3)
        if d == 1:
            f[:] = 2.0  # symmetric fronts: both sides of an axis equal
        xs, ys = axis(shape[2], lo, hi), axis(shape[1], lo, hi)
        zs = axis(nz, lo, hi) if nz > 1 else None
        for src in (np.array([f.size // 2], dtype=np.int64), np.array([0, f.size - 1], dtype=np.int64)):
            t0 = np.linspace(0.0, 0.3, src.size) * float(np.ptp(xs))
            ref = O.solve_rect(f, xs, ys, zs, src, t0=t0).reshape(shape)
            fd = torch.from_numpy(f if nz > 1 else f[0]).cuda()
            got = gpu.solve_rect(fd, xs, ys, zs, torch.from_numpy(src), t0=torch.from_numpy(t0),
                                 delta=float(np.ptp(xs)) / 20, tile=tile if tz > 1 else tile[:2])
            got = got.cpu().numpy().reshape(shape)
            assert np.array_equal(got.view(np.uint64), ref.view(np.uint64)), (shape, d)


@pytest.mark.parametrize("nx", [1, 2, 3, 4, 5, 7, 8, 63, 65, 257])
def test_parent_rows(gpu, O, nx):
    """The parent record takes four points of a row at a time: row lengths around
    multiples of four, constant media (ties everywhere), and a batch whose chunks
    of points start inside a row."""
    rng = np.random.default_rng(nx)
    fields, srcs = [], []
    for i, shape in enumerate(((2, 9, nx), (5, 3, nx), (2, 1, nx), (4, 31, nx))):
        f = W.random_field(shape, rng, 0.5, 2.0) if i % 2 else np.full(shape, 2.0)
        fields.append(f)
        srcs.append(np.unique(rng.integers(0, f.size, 2)).astype(np.int64))
    dev = [torch.from_numpy(f).cuda() for f in fields]
    ts, pars = gpu.solve_batched(dev, 1.0, [torch.from_numpy(s) for s in srcs], parents=True, delta=0.5, tile=(8, 8, 8))
    for f, d, s, t, p in zip(fields, dev, srcs, ts, pars):
        ref = O.fmm(f, 1.0, s)
        par = O.parents(ref, s).reshape(-1)
        assert np.array_equal(p.cpu().numpy().reshape(-1), par), f.shape
        alone = gpu.parents_of(torch.from_numpy(ref.reshape(d.shape)).cuda(), torch.from_numpy(s))
        assert np.array_equal(alone.cpu().numpy().reshape(-1), par), f.shape


@pytest.mark.parametrize("tile", TILES)
def test_adjoint_tile_edges(gpu, O, tile):
    rng = np.random.default_rng(100 + sum(tile))
    tx, ty, tz = tile
    for d in (-1, 0, 1):
        nz = 1 if tz == 1 else max(tz + d, 2)
        shape = (nz, max(2 * ty - d, 2), max(2 * tx + d, 2))
        f = W.random_field(shape, rng, 0.5, 5.0, block=2)
        src = np.unique(rng.integers(0, f.size, 3)).astype(np.int64)
        t = O.fmm(f, 1.0, src)
        par = O.parents(t, src)
        g = rng.standard_normal(shape)
        g[rng.random(shape) < 0.5] = 0.0
        ref = O.adjoint(t, par, f, 1.0, g).reshape(shape)
        sq = (lambda a: a) if tz > 1 else (lambda a: a.reshape(shape)[0])
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(sq(a.reshape(shape)))).cuda()
        for kw in (dict(), dict(delta=1.0, lookahead=4)):
            got = gpu.adjoint(dev(f), 1.0, dev(t), dev(par), dev(g), tile=tile if tz > 1 else tile[:2], **kw)
            got = got.cpu().numpy().reshape(shape)
            err = np.max(np.abs(got - ref)) / np.max(np.abs(ref))
            assert err <= 1e-12, (shape, kw, err)
