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
