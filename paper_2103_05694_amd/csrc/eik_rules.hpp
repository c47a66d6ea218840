// Rules the kernels decide by that are plain arithmetic: also compiled for the
// host, where they are checked at their limits.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define EIK_RULE __host__ __device__ __forceinline__
#else
#define EIK_RULE inline
#endif

namespace eik {

// Launches of so few tiles that a run's own time decides take a workgroup per tile
// (eik_block.hpp) instead of a wave per tile: `total` tiles, `most` of them in one
// problem.  A run takes about half as long with all of a tile's points at once; a
// wave evaluates fewer points and a compute unit holds five to ten of them.  How
// much fewer depends on the medium: least in random speeds with a source inside
// (below "random"), most for a front through layers ("layered"), so the lines lie
// where neither loses more than the other gains.  Measured, wave / workgroup per
// tile, whole calls in ms:
//  * solves in 3D, 16x8x8, random and layered: 1 tile 0.18 / 0.12, 384 tiles 3.05 /
//    1.90 and 1.45 / 1.17, 1000 tiles 3.65 / 3.20 and 1.87 / 1.65, 1584 tiles 4.07 /
//    4.21 and 2.21 / 2.43; 400 problems of 4 tiles 1.20 / 0.79 and 0.47 / 0.45, 200 of
//    12 1.57 / 1.73 and 0.66 / 1.02, 30 of 64 2.08 / 2.49 and 1.00 / 1.06.  Tiles of 256
//    points or fewer gain little beyond one (8x8x4: 1 tile 0.104 / 0.088, 256 tiles
//    0.82 / 0.77).
//  * solves in 2D, where a front crosses a tile in twice the passes, 32x32: 1 tile
//    0.158 / 0.124, 1000 problems of one 0.27 / 0.26; 12 tiles of one problem 0.52 / 0.49
//    and 0.31 / 0.39; 100 problems of 4 tiles 0.64 / 0.49 and 0.31 / 0.31, 400 of 4 0.83 /
//    0.72 and 0.45 / 0.54.
//  * rectilinear solves, whose operator is the longest: 1 tile 0.46 / 0.32 (2D) and
//    0.79 / 0.46 (3D), 4 tiles of 8x8x8 1.18 / 1.06, 12 tiles of 16x8x8 7.2 / 6.1 (random)
//    and 0.64 / 0.63 (layered), 24 tiles 1.10 / 1.33 (layered).
//  * adjoints, which evaluate a point once: 16x8x8 1 tile 0.125 / 0.080, 32 tiles 1.22 /
//    0.89 and 0.35 / 0.36, 512 tiles 3.13 / 2.37 and 1.43 / 1.25, 200 problems of 4 0.56 /
//    0.51 and 0.34 / 0.31, 400 of 4 0.62 / 0.74 and 0.40 / 0.49; 8x8x8 12 tiles 0.31 / 0.29
//    and 0.175 / 0.170, 32 tiles 0.36 / 0.33 and 0.22 / 0.25; 64x4x4 4 tiles 1.13 / 0.92 and
//    0.19 / 0.27; 32x32 4 tiles 0.24 / 0.21 and 0.18 / 0.22, 100 problems of 4 0.38 / 0.36
//    and 0.31 / 0.30, 200 of 4 0.44 / 0.48 and 0.38 / 0.42.
template <int TX, int TY, int TZ>
struct FewTiles {
    static constexpr int NP = TX * TY * TZ;
    static constexpr bool kSquare = TX == 32 && TY == 32;
    // whether the kernels are there for this shape at all
    static constexpr bool kSolve = NP >= 256, kAdjoint = NP >= 512;
    static EIK_RULE bool solve(int64_t most, int64_t total) {
        if (TZ > 1 && NP >= 512) return total <= (most <= 16 ? 1600 : 1024);
        if (kSquare) return total <= 900 && (most == 1 || (most <= 9 && total >= 100));
        return kSolve && most == 1 && total <= 512;
    }
    static EIK_RULE bool rect(int64_t total) {
        return kSolve && total <= (TZ > 1 && NP >= 512 ? (NP >= 1024 ? 12 : 8) : 1);
    }
    static EIK_RULE bool adjoint(int64_t most, int64_t total) {
        if (TZ >= 8) return total <= 800 && (NP >= 1024 || most <= 16);
        if (kSquare && most > 1) return most <= 9 && total >= 100 && total <= 400;
        return kAdjoint && most == 1 && total <= 512;
    }
};

// Whether the cells of a tile that lies wholly in the grid, and of its face halos,
// can be addressed by 32-bit byte offsets from the corner of the halo (one point
// before the tile along each axis) in an array of doubles.  The furthest along
// are the far corners of the z+ and y+ halos, TZ + 1 planes, TY rows and TX points
// and TZ planes, TY + 1 rows and TX points from it; the bound covers both.
template <int TX, int TY, int TZ>
EIK_RULE bool offsets_fit_32(int64_t nx, int64_t plane) {
    const int64_t last = (TZ > 1 ? (TZ + 1) * plane : 0) + (TY + 1) * nx + TX + 1;
    return last < (1ll << 29);
}

// Index of the last of n ascending values that are not above a bound (the first
// one is not), by 64 probes at once: count(first, step, n) tells how many of the
// values first + i * step (i < 64, i * step < n) are not above it.  One round up
// to 64 values, two up to 4096, three up to 262144.
template <class Count>
EIK_RULE int last_not_above(int n, Count count) {
    int first = 0;
    while (n > 64) {
        const int step = (n + 63) / 64;
        const int at = (count(first, step, n) - 1) * step;
        first += at;
        n = n - at < step ? n - at : step;
    }
    return first + count(first, 1, n) - 1;
}

// Buckets from the current one on that a claim may take work from: `lookahead`
// beyond the current one, and for a worker that has found nothing in kPatience
// polls kWide of them, unless the caller wants the window kept (`strict`).
constexpr int kWide = 17, kPatience = 3;
EIK_RULE int claim_window(int lookahead, bool strict, long long idle_polls) {
    const int own = lookahead + 1;
    return strict || idle_polls < kPatience || own > kWide ? own : kWide;
}

// When a worker that waits for work gives up (an internal error: the launch can
// make no progress any more).  It looks now and then at a word that every end of
// a run changes, handed on or not, and gives up once that has stood still for
// kStallTicks, or as soon as another worker has, so that one expiry ends the
// launch.  Time alone would also pass while the whole process is off the device,
// so it takes kStallLooks looks as well (a tenth of a second of polling or more).
constexpr uint64_t kStallTicks = 1400000000ull;  // 14 s of the 100 MHz clock
constexpr uint32_t kStallLooks = 4096;
struct StallWatch {
    uint64_t seen = 0, since = 0;
    uint32_t looks = 0;  // since `seen` was first seen (0: not looked yet)
    EIK_RULE bool gives_up(uint64_t progress, bool another_did, uint64_t now) {
        if (another_did) return true;
        if (looks == 0 || progress != seen) {
            seen = progress;
            since = now;
            looks = 1;
            return false;
        }
        if (looks < kStallLooks) ++looks;
        return looks == kStallLooks && now - since > kStallTicks;
    }
};

}  // namespace eik
