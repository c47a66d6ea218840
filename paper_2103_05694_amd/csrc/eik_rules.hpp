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

}  // namespace eik
