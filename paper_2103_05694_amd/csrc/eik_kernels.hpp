// Forward kernels: per-solve reset, source placement, finalisation, the
// upwind-parent record and the residual; the solvers themselves are in
// eik_sweep.hpp and eik_block.hpp.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "eik_op.hpp"
#include "eik_rules.hpp"
#include "eik_sched.hpp"

namespace eik {

// One problem of a (possibly batched) launch.
struct Prob {
    int32_t nx, ny, nz;      // points per axis
    int32_t ntx, nty, ntz;   // tiles per axis
    int64_t pt_off;          // first point in the packed arrays
    int32_t tile_off;        // first global tile id
    int32_t kind;            // 0 speed (q = h/v), 1 slowness (q = h*s)
    double h;
};

// Problem table of a launch.  A single problem travels by value in the kernel
// arguments (no upload, no host synchronisation); batches read the device table.
struct ProbTable {
    const Prob* probs;       // device table, used when nprob > 1
    const int64_t* src_off;  // device source offsets, used when nprob > 1
    int nprob;
    int most_tiles;          // of one problem
    Prob p0;                 // the problem when nprob == 1
    int64_t nsrc0;           // its source count
};

struct SolveArgs {
    ProbTable pt;
    const double* field;
    double* t;
    uint64_t* tkey;          // [ntiles] pending requeue key (bits of a positive double)
    const double* work_ref;  // NULL, or the final times: classify every evaluation
    // rectilinear grids (OP 4): reciprocal spacings per axis and index, laid
    // out [wm_x (nx), wp_x (nx), wm_y (ny), wp_y (ny), wm_z (nz), wp_z (nz)]
    const double* rw;
    int warm;                // t holds a caller's upper bound (warm start)
    Sched s;
};

__device__ __forceinline__ Prob prob_of_tile(const ProbTable& T, int tile) {
    if (T.nprob == 1) return T.p0;
    int lo = 0, hi = T.nprob - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (T.probs[mid].tile_off <= tile) lo = mid; else hi = mid - 1;
    }
    return T.probs[lo];
}

__device__ __forceinline__ Prob prob_of_point(const ProbTable& T, long long g) {
    if (T.nprob == 1) return T.p0;
    int lo = 0, hi = T.nprob - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (T.probs[mid].pt_off <= g) lo = mid; else hi = mid - 1;
    }
    return T.probs[lo];
}

__device__ __forceinline__ Prob prob_of_source(const ProbTable& T, long long g) {
    if (T.nprob == 1) return T.p0;
    int lo = 0, hi = T.nprob - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (T.src_off[mid] <= g) lo = mid; else hi = mid - 1;
    }
    return T.probs[lo];
}

__device__ __forceinline__ double field_q(double f, double h, int kind, bool& ok) {
    double q = kind == 0 ? h / f : h * f;
    double c = q * q;
    ok = (f > 0.0) && (f < inf64()) && (c > 0.0) && (c < inf64());
    return q;
}

// ---------------------------------------------------------------------------
// per-solve set-up
// ---------------------------------------------------------------------------

// Clears tile states and requeue keys, the window, counters and flags, and (t not
// NULL) sets t to +inf at every point: a solve starts from the upper bound +inf
// everywhere.  When the previous solve on this workspace ended abnormally
// (`poisoned`), or the caller asks for it (`force_wipe`: memory whose contents
// are not known yet), it also re-initialises the rings so no stale slot can be
// taken for a new item.
__global__ void k_reset(Sched s, uint64_t* tkey, int ntiles, long long ring_words, int force_wipe, double* t,
                        long long npts) {
    const bool wipe = force_wipe || __hip_atomic_load(s.poisoned, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
    const long long stride = (long long)gridDim.x * blockDim.x;
    const long long i0 = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    for (long long i = i0; i < ntiles; i += stride) {
        s.tstate[i] = 0u;
        tkey[i] = kInfBits;
    }
    if (wipe) {
        // cell i of every ring starts free for position i (lap 0)
        const long long cap = (long long)s.cap_mask + 1;
        for (long long i = i0; i < ring_words; i += stride) s.items[i] = (uint64_t)(i % cap) << 32;
        // head = tail = 0; count word = bias (0 queued, 0 running)
        for (long long i = i0; i < (long long)kPendWord; i += stride)
            s.ctr[i] = (i % kCtrStride) == kCrWord ? (uint32_t)kCountBias : 0u;
    }
    if (i0 < kCounters) s.counters[i0] = 0ull;
    if (i0 < kShards) *pend_word(s, (int)i0) = 0ull;
    if (i0 == 0) {
        if (s.timeline) {
            s.timeline[0] = wall_clock64();
            s.timeline[1] = 0ull;
        }
        *s.cur = 0;
        *s.flags = 0u;
    }
    if (t)
        for (long long i = i0; i < npts; i += stride) t[i] = inf64();
}

template <int TX, int TY, int TZ>
__device__ __forceinline__ uint32_t tile_of_point(const Prob& P, int64_t local) {
    int64_t x = local % P.nx, y = (local / P.nx) % P.ny, z = local / ((int64_t)P.nx * P.ny);
    return (uint32_t)(P.tile_off + ((z / TZ) * P.nty + (y / TY)) * P.ntx + (x / TX));
}

__device__ __forceinline__ bool src_ok(const Prob& P, int64_t idx, double t0) {
    int64_t n = (int64_t)P.nx * P.ny * P.nz;
    return idx >= 0 && idx < n && t0 >= 0.0 && t0 < inf64() && !signbit(t0);
}

// Writes each source as -t0 (the sign bit marks a fixed point during the solve;
// min over duplicates through the signed image, where -0.0 is the smallest),
// marks its tile (S) and queues it.
template <int TX, int TY, int TZ>
__global__ void k_src_place(ProbTable T, const int64_t* src_idx, const double* src_t0, long long nsrc,
                            double* t, Sched s) {
    long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (g == 0) *s.poisoned = 0;  // the reset before this kernel has wiped the rings
    if (g >= nsrc) return;
    const Prob P = prob_of_source(T, g);
    int64_t idx = src_idx[g];
    double t0 = src_t0 ? src_t0[g] : 0.0;
    if (!src_ok(P, idx, t0)) {
        set_flag(s, kFlagBadSrc);
        return;
    }
    long long* ti = (long long*)(t + P.pt_off + idx);
    __hip_atomic_fetch_min(ti, (long long)as_u64(-t0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t tile = tile_of_point<TX, TY, TZ>(P, idx);
    uint32_t old = __hip_atomic_fetch_or(s.tstate + tile, kQ | kS, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!(old & kQ)) activate_push(s, tile, t0);
}

// Restores +t0 at the sources.
__global__ void k_src_unsign(ProbTable T, const int64_t* src_idx, const double* src_t0, long long nsrc,
                             double* t) {
    long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= nsrc) return;
    const Prob P = prob_of_source(T, g);
    int64_t idx = src_idx[g];
    double t0 = src_t0 ? src_t0[g] : 0.0;
    if (!src_ok(P, idx, t0)) return;
    double* ti = t + P.pt_off + idx;
    *ti = fabs(*ti);
}

// ---------------------------------------------------------------------------
// warm start: resume from an upper bound of the solution
// ---------------------------------------------------------------------------

// Checks a caller-supplied starting state and records each tile's smallest
// value (bits of a non-negative double; kInfBits when the tile is all +inf).
// A value that is NaN or has its sign bit set (the solver's source marker) is
// not a valid upper bound: it raises kFlagBadStart and is replaced by +inf, so
// the solve still runs on a valid state.
template <int TX, int TY, int TZ>
__global__ void k_warm_prep(ProbTable T, int ntiles, double* t, uint64_t* tile_min, Sched s) {
    __shared__ unsigned long long s_m;
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const Prob P = prob_of_tile(T, tile);
        const int tl = tile - P.tile_off;
        const int tx = tl % P.ntx, ty = (tl / P.ntx) % P.nty, tz = tl / (P.ntx * P.nty);
        if (threadIdx.x == 0) s_m = kInfBits;
        __syncthreads();
        unsigned long long m = kInfBits;
        for (int i = threadIdx.x; i < TX * TY * TZ; i += blockDim.x) {
            const int lx = i % TX, ly = (i / TX) % TY, lz = i / (TX * TY);
            const int x = tx * TX + lx, y = ty * TY + ly, z = tz * TZ + lz;
            if (x < P.nx && y < P.ny && z < P.nz) {
                double* p = t + P.pt_off + ((int64_t)z * P.ny + y) * P.nx + x;
                const double v = *p;
                if (v != v || signbit(v)) {
                    set_flag(s, kFlagBadStart);
                    *p = inf64();
                } else if (as_u64(v) < m) {
                    m = as_u64(v);
                }
            }
        }
        if (m != kInfBits) atomicMin(&s_m, m);
        __syncthreads();
        if (threadIdx.x == 0) tile_min[tile] = s_m;
        __syncthreads();
    }
}

// Queues every tile that has a finite value in itself or in a face neighbour
// (any other tile can only change once a neighbour lowers its face, which
// activates it), keyed by the smallest of those values.  Tiles already queued
// (the source tiles) are left alone.  Their state words were cleared by the
// reset, so every first run relaxes all of its points.
__global__ void k_warm_push(ProbTable T, int ntiles, const uint64_t* tile_min, Sched s) {
    for (int tile = blockIdx.x * blockDim.x + threadIdx.x; tile < ntiles; tile += gridDim.x * blockDim.x) {
        const Prob P = prob_of_tile(T, tile);
        const int tl = tile - P.tile_off;
        const int t3[3] = {tl % P.ntx, (tl / P.ntx) % P.nty, tl / (P.ntx * P.nty)};
        const int lim[3] = {P.ntx, P.nty, P.ntz};
        uint64_t key = tile_min[tile];
        for (int f = 0; f < 6; ++f) {
            int nt[3] = {t3[0], t3[1], t3[2]};
            nt[f >> 1] += (f & 1) ? 1 : -1;
            if (nt[f >> 1] < 0 || nt[f >> 1] >= lim[f >> 1]) continue;
            const uint64_t k = tile_min[P.tile_off + (nt[2] * P.nty + nt[1]) * P.ntx + nt[0]];
            if (k < key) key = k;
        }
        if (key == kInfBits) continue;
        const uint32_t old = __hip_atomic_fetch_or(s.tstate + tile, kQ, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!(old & kQ)) activate_push(s, (uint32_t)tile, as_f64(key));
    }
}

// ---------------------------------------------------------------------------
// shared by the tile kernels
// ---------------------------------------------------------------------------

__device__ __forceinline__ double hload(const double* p) {
    // Halo cells belong to tiles other workgroups may be writing right now.
    uint64_t u = __hip_atomic_load((const uint64_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return fabs(as_f64(u));
}

__device__ __forceinline__ void tstore(double* p, double v) {
    __hip_atomic_store((uint64_t*)p, as_u64(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Minimum over the 64 lanes of a wave (every lane gets it).
__device__ __forceinline__ double wave_min(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = nmin(v, __shfl_xor(v, off));
    return v;
}

// Adds a worker's statistics to the launch's: [0..3] phase times, [4] visits,
// [5] point updates, [6] passes, [7] hand-offs.  Single lane.
__device__ __forceinline__ void flush_stats(const Sched& S, const unsigned long long* st) {
    auto add = [&](int i, unsigned long long v) {
        __hip_atomic_fetch_add(S.counters + i, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    for (int i = 0; i < 4; ++i) add(5 + i, st[i]);
    add(10, 1ull);
    add(12, st[7]);
    add(0, st[4]);
    add(1, st[5]);
    add(2, st[6]);
    if (S.timeline)
        __hip_atomic_fetch_max(S.timeline + 1, (unsigned long long)wall_clock64(), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------------------
// residual of a solution (the error metric of Table "tab:error")
// ---------------------------------------------------------------------------

__global__ void k_fill_u8(long long n, uint8_t* a, uint8_t v) {
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) a[i] = v;
}

// Clears the residual accumulators: out[0] count, out[1] max, out[2] flags.
__global__ void k_clear_residual(unsigned long long* out) {
    if (threadIdx.x < 3) out[threadIdx.x] = 0ull;
}

__global__ void k_mark_points(const int64_t* idx, long long n, long long npts, uint8_t* mask) {
    const long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n) return;
    const int64_t i = idx[g];
    if (i >= 0 && i < npts) mask[i] = 1;
}

// Counts the non-source points whose time differs from the operator applied
// to their final neighbours, and the largest relative difference (bits of a
// non-negative double, atomic max): out[0] count, out[1] max.  Field values
// that are not positive and finite raise the domain flag.
template <int OP>
__global__ void k_residual(Prob P, const double* field, const double* t, const uint8_t* fixed,
                           unsigned long long* out, uint32_t* flags) {
    const long long n = (long long)P.nx * P.ny * P.nz;
    const long long stride = (long long)gridDim.x * blockDim.x;
    unsigned long long cnt = 0, worst = 0;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        if (fixed[i]) continue;
        bool ok;
        const double q = field_q(field[i], P.h, P.kind, ok);
        if (!ok) {
            __hip_atomic_fetch_or(flags, kFlagDomain, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            continue;
        }
        const long long x = i % P.nx, y = (i / P.nx) % P.ny, z = i / ((long long)P.nx * P.ny);
        const long long sy = P.nx, sz = (long long)P.nx * P.ny;
        double lo = x > 0 ? t[i - 1] : inf64(), hi = x < P.nx - 1 ? t[i + 1] : inf64();
        const double ax = lo < hi ? lo : hi;
        lo = y > 0 ? t[i - sy] : inf64();
        hi = y < P.ny - 1 ? t[i + sy] : inf64();
        const double ay = lo < hi ? lo : hi;
        double az = inf64();
        if (P.nz > 1) {
            lo = z > 0 ? t[i - sz] : inf64();
            hi = z < P.nz - 1 ? t[i + sz] : inf64();
            az = lo < hi ? lo : hi;
        }
        const double r = apply_op<OP>(ax, ay, az, q);
        const double ti = t[i];
        if (r != ti) {
            ++cnt;
            const unsigned long long rb = as_u64(fabs(r - ti) / fabs(ti)) & ~kSignBit;
            if (rb > worst) worst = rb;
        }
    }
    if (cnt) __hip_atomic_fetch_add(out, cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (worst) __hip_atomic_fetch_max(out + 1, worst, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------------------
// upwind-parent record
// ---------------------------------------------------------------------------

// The parent byte of a point with value t from its neighbours.  Reads |t|: a set
// sign bit marks a source while the solve's encoding is still in place (then
// bit 7 is written).  A neighbour off the grid is given as the point itself: it
// is then no parent, and not the smaller of two of which the other is.
__device__ __forceinline__ uint32_t parent_byte(double t, double xm, double xp, double ym, double yp, double zm,
                                                double zp) {
    auto code = [&](double l, double r) { return fmin(fabs(l), fabs(r)) < t ? (fabs(l) <= fabs(r) ? 1u : 2u) : 0u; };
    const uint32_t b = code(xm, xp) | code(ym, yp) << 2 | code(zm, zp) << 4;
    return signbit(t) ? 0x80u : b;
}

// Parents of all points of the launch, four consecutive points a thread.  Bound
// by memory (9 B per point once the neighbours hit the caches) only if the
// index arithmetic stays small: a block takes kParChunk consecutive points and
// finds their problem once, and a thread divides once for four points, whose
// rows it reads as vectors (512x512x256: 498 us with a search and three 64-bit
// divisions per point, 345 us point by point without them).  With UNSIGN it also
// restores +t0 at the sources; other threads read those values as |t|.
constexpr int kParThreads = 256, kParSteps = 4, kParChunk = 4 * kParThreads * kParSteps;
template <bool UNSIGN>
__global__ void __launch_bounds__(kParThreads) k_parents(ProbTable T, long long npts_total, double* t,
                                                         uint8_t* par) {
    // one point by the general route
    auto single = [&](long long g) {
        const Prob Q = prob_of_point(T, g);
        const int64_t i = g - Q.pt_off, row = i / Q.nx, sy = Q.nx, sz = (int64_t)Q.nx * Q.ny;
        const int x = (int)(i - row * Q.nx), y = (int)(row % Q.ny), z = (int)(row / Q.ny);
        const double* at = t + g;
        const double c = at[0];
        if (UNSIGN && signbit(c)) t[g] = fabs(c);
        par[g] = (uint8_t)parent_byte(c, at[x > 0 ? -1 : 0], at[x < Q.nx - 1 ? 1 : 0], at[y > 0 ? -sy : 0],
                                      at[y < Q.ny - 1 ? sy : 0], at[z > 0 ? -sz : 0], at[z < Q.nz - 1 ? sz : 0]);
    };
    for (long long c0 = (long long)blockIdx.x * kParChunk; c0 < npts_total; c0 += (long long)gridDim.x * kParChunk) {
        const long long c1 = c0 + kParChunk < npts_total ? c0 + kParChunk : npts_total;
        const Prob P = prob_of_point(T, c0);
        const int64_t n = (int64_t)P.nx * P.ny * P.nz, sy = P.nx, sz = (int64_t)P.nx * P.ny;
        // whole chunk in one problem, indices in 32 bits
        const bool plain = c1 - P.pt_off <= n && n < (1ll << 31);
#pragma unroll
        for (int s = 0; s < kParSteps; ++s) {
            const long long g = c0 + 4 * (s * kParThreads + (int)threadIdx.x);
            if (g >= c1) continue;
            const uint32_t i = (uint32_t)(g - P.pt_off), row = i / (uint32_t)P.nx;
            const int x = (int)(i - row * (uint32_t)P.nx);
            if (!plain || g + 4 > c1 || x + 4 > P.nx) {  // the four points are not of one row
                for (long long k = g; k < g + 4 && k < c1; ++k) single(k);
                continue;
            }
            const int z = (int)(row / (uint32_t)P.ny), y = (int)(row - (uint32_t)z * (uint32_t)P.ny);
            const double* at = t + g;
            double c[4], ym[4], yp[4], zm[4], zp[4];
            __builtin_memcpy(c, at, 32);
            const double xl = at[x > 0 ? -1 : 0], xr = at[x + 4 < P.nx ? 4 : 3];
            __builtin_memcpy(ym, at + (y > 0 ? -sy : 0), 32);
            __builtin_memcpy(yp, at + (y < P.ny - 1 ? sy : 0), 32);
            __builtin_memcpy(zm, at + (z > 0 ? -sz : 0), 32);
            __builtin_memcpy(zp, at + (z < P.nz - 1 ? sz : 0), 32);
            uint32_t b = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                b |= parent_byte(c[k], k > 0 ? c[k - 1] : xl, k < 3 ? c[k + 1] : xr, ym[k], yp[k], zm[k], zp[k]) << (8 * k);
            __builtin_memcpy(par + g, &b, 4);
            if (UNSIGN && (b & 0x80808080u)) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (signbit(c[k])) t[g + k] = fabs(c[k]);
            }
        }
    }
}

// Marks sources in a parent record computed from final (unsigned) times.
__global__ void k_parents_mark_src(ProbTable T, const int64_t* src_idx, long long nsrc, uint8_t* par) {
    long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= nsrc) return;
    const Prob P = prob_of_source(T, g);
    int64_t idx = src_idx[g];
    if (idx < 0 || idx >= (int64_t)P.nx * P.ny * P.nz) return;
    par[P.pt_off + idx] = 0x80;
}

}  // namespace eik
