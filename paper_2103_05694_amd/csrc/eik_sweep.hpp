// The persistent forward solver of all but small launches: one wave per tile, and
// as many waves (tiles in flight) on a compute unit as its LDS holds tiles.
//
// A wave claims the approximately earliest active tile (eik_sched.hpp), stages its
// times, the 1-cell halo and the per-point constants in LDS, applies the update operator to dirty points until nothing
// in the tile changes, writes the lowered points back and activates the face
// neighbours whose halo changed (the paper's asynchronous marching method with
// a tile as the unit of work; Theorem 1 makes every order reach the same bits).
//
// In-tile order.  Each lane walks one column of the tile along x (with fewer
// than 64 columns, 64 / columns lanes share one, evenly spaced along it), and
// lane (y, z) is y + z steps behind lane (0, 0).  The points visited at one
// step (a level) are then x + y + z = const: no two of them are neighbours, and
// each comes after its three upwind neighbours of the octant swept.  So one
// sweep settles a front crossing the tile in that octant with about one
// operator evaluation per point, where evaluating every dirty point at once
// (Jacobi order) re-evaluates a point each time one of its neighbours drops.
// A level needs no barrier: the wave runs in lockstep and its LDS accesses are
// performed in order.
//
// What bounds it.  The bytes it must move (16 per point) are a hundredth of its
// time.  On a large grid with one source the front's chain of tiles does: a level
// takes about 0.55 us, almost all of it the serial chain of the operator's FP64
// instructions (10 cycles each), staging and publishing a tile about 10 us, and
// most waves wait for the front (13601x2801: 300 us per run waiting, 42 us
// running).  With many problems at once the waves are busy and the FP64 issue
// and the LDS capacity (6 tiles of 16x8x8 a compute unit) bound it.  A workgroup
// of 512 or 1024 threads per tile, Jacobi passes with a barrier each and rings
// not split into shards took, for the whole call: 512x512x256 layered, 16x8x8
// tiles, 24.7 ms against 11.7; 4096x4096, 16 sources, 32x32 tiles, 12.4 against
// 6.4 ms; 13601x2801, 37.0 against 30.0 ms; 32 problems of 256x256x128 (forward
// and adjoint) 139 against 58 ms.  (On launches of few tiles that form, with the
// shards, is the better one: eik_block.hpp.)  More waves than tiles in LDS
// (waiting for a free one) made the batch 4% faster and everything else 5%
// slower, and is not done.
//
// Only dirty points are evaluated.  A lane keeps the dirty bits of the points
// it visits next in a register, bit i for the point i levels ahead.  In sweep
// order a lowered point's neighbour ahead along any axis is the very next
// point of the lane that visits it, and a neighbour behind the last one its
// lane will visit (NPT - 1 levels ahead), so marking neighbours is two bit sets
// from lane masks that the comparisons leave in scalar registers.  The run ends
// when no lane has a bit left; the octant is chosen again after each sweep, from
// the sides of the points still dirty that their smaller neighbours are on.
#pragma once

#include <type_traits>

#include "eik_kernels.hpp"

namespace eik {

template <int TX, int TY, int TZ>
struct SweepCfg {
    static constexpr bool D3 = TZ > 1;
    static constexpr int SY = TX + 2;
    static constexpr int SZ = (TX + 2) * (TY + 2);
    static constexpr int HZ = D3 ? TZ + 2 : 1;
    static constexpr int ZOFF = D3 ? 1 : 0;
    static constexpr int NLDS = SZ * HZ;
    static constexpr int NP = TX * TY * TZ;
    static constexpr int NPT = NP / 64;           // points per lane, and levels per cycle
    static constexpr int NCOL = TY * TZ;          // columns along x
    static constexpr int SPAN = TX + TY + TZ - 2; // levels of one sweep corner to corner; the octant is
                                                  // chosen again after each
    static constexpr int NF = D3 ? 6 : 4;
    // waves (tiles in flight) per workgroup: what the 160 KB of LDS of a
    // compute unit hold, one workgroup each, at most 16
    static constexpr int BYTES = 8 * NLDS + 8 * NP + 2 * NP;
    static constexpr int FIT = (160 * 1024 - 1024) / (BYTES + 16 * (TX + TY + TZ) + 80);
    static constexpr int W = FIT < 16 ? FIT : 16;
    static constexpr int WPE = (W + 3) / 4;                            // waves per SIMD
    static_assert(NCOL <= 64 && 64 % NCOL == 0, "whole columns per wave");
    static_assert((TX & (TX - 1)) == 0 && (TY & (TY - 1)) == 0 && (TZ & (TZ - 1)) == 0, "powers of two");
    static_assert(NPT >= 2, "two lanes of one column must never visit neighbouring points");
    __device__ static constexpr int lds(int lx, int ly, int lz) {
        return (lz + ZOFF) * SZ + (ly + 1) * SY + (lx + 1);
    }
    // Lanes whose column (yy, zz) is not the first (side 0) or last (side 1) along an axis.
    static constexpr unsigned long long inner(int axis, int side) {
        unsigned long long m = 0;
        for (int l = 0; l < 64; ++l) {
            const int v = axis == 1 ? l % TY : (l / TY) % TZ, n = axis == 1 ? TY : TZ;
            if (side ? v < n - 1 : v > 0) m |= 1ull << l;
        }
        return m;
    }
    // Points p = lane + 64 j and lanes: a step j moves every lane by the same
    // (DY, DZ) rows and planes (DX points where a row is longer than the wave).
    // Byte of point p in an array where the points of a lane (p = lane + 64 j) are adjacent.
    __device__ static constexpr int mine(int p) { return (int)((((unsigned)p & 63u) * NPT) | ((unsigned)p >> 6)); }
    __device__ static constexpr int jx(int j) { return TX > 64 ? (64 * j) % TX : 0; }
    __device__ static constexpr int jy(int j) { return (64 * j / TX) % TY; }
    __device__ static constexpr int jz(int j) { return 64 * j / (TX * TY); }
};

// Orders this wave's LDS accesses for the compiler (the hardware performs a
// wave's LDS accesses in order).
__device__ __forceinline__ void wave_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// The problem a tile belongs to, found by the wave together: one load of up to
// 64 first tile ids per round instead of a binary search of dependent loads.
__device__ __forceinline__ Prob wave_prob_of_tile(const ProbTable& T, int tile) {
    if (T.nprob == 1) return T.p0;
    const int lane = threadIdx.x & 63;
    const int k = last_not_above(T.nprob, [&](int first, int step, int n) {
        const long long i = (long long)lane * step;
        return (int)__popcll(__ballot(i < n && T.probs[first + i].tile_off <= tile));
    });
    return T.probs[uni(k)];
}

// Cell c of face f (x-, x+, y-, y+, z-, z+) of a tile: the tile point on the
// face and the distance in LDS to the halo cell across it.
template <int TX, int TY, int TZ>
struct Face {
    int lx, ly, lz;
    __device__ static constexpr int cells(int f) { return f < 2 ? TY * TZ : (f < 4 ? TX * TZ : TX * TY); }
    __device__ static constexpr int out(int f) {
        using C = SweepCfg<TX, TY, TZ>;
        return (f & 1 ? 1 : -1) * (f < 2 ? 1 : (f < 4 ? C::SY : C::SZ));
    }
    __device__ __forceinline__ Face(int f, int c) {
        const int side = f & 1;
        if (f < 2) {
            lx = side ? TX - 1 : 0; ly = c % TY; lz = c / TY;
        } else if (f < 4) {
            lx = c % TX; ly = side ? TY - 1 : 0; lz = c / TX;
        } else {
            lx = c % TX; ly = c / TX; lz = side ? TZ - 1 : 0;
        }
    }
    __device__ __forceinline__ int lds() const { return SweepCfg<TX, TY, TZ>::lds(lx, ly, lz); }
    __device__ __forceinline__ int point() const { return (lz * TY + ly) * TX + lx; }
};

// Smallest value over the wave (unsigned), in registers: row shifts within 16
// lanes, then the two row broadcasts, leave it in lane 63.
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
#define EIK_DPP_MIN(ctrl, rows)                                                                        \
    {                                                                                                  \
        const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, ctrl, rows, 0xF, false); \
        v = o < v ? o : v;                                                                             \
    }
    EIK_DPP_MIN(0x111, 0xF)  // row_shr:1
    EIK_DPP_MIN(0x112, 0xF)  // row_shr:2
    EIK_DPP_MIN(0x114, 0xF)  // row_shr:4
    EIK_DPP_MIN(0x118, 0xF)  // row_shr:8
    EIK_DPP_MIN(0x142, 0xA)  // row_bcast:15 into rows 1 and 3
    EIK_DPP_MIN(0x143, 0xC)  // row_bcast:31 into rows 2 and 3
#undef EIK_DPP_MIN
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// The same for 64 bits: the smallest high half, then the smallest low half of the
// lanes that have it, which is mostly one lane.
__device__ __forceinline__ uint64_t wave_min_u64(uint64_t v) {
    const uint32_t hi = wave_min_u32((uint32_t)(v >> 32));
    const unsigned long long who = __ballot((uint32_t)(v >> 32) == hi);
    uint32_t lo;
    if ((who & (who - 1)) == 0)
        lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, __ffsll((long long)who) - 1);
    else
        lo = wave_min_u32((uint32_t)(v >> 32) == hi ? (uint32_t)v : ~0u);
    return ((uint64_t)hi << 32) | lo;
}

// One wave's tile in LDS.
template <int TX, int TY, int TZ, int OP>
struct SweepTile {
    using C = SweepCfg<TX, TY, TZ>;
    double t[C::NLDS];
    double q[C::NP];
    // rectilinear grids: reciprocal spacings [x- | x+ | y- | y+ | z- | z+] over the tile's coordinates
    double wx[OP == 4 ? 2 * (TX + TY + TZ) : 1];
    unsigned long long stat[9];       // as in Block
    alignas(8) uint8_t dirty[C::NP];  // marks carried into the next sweep (these two are cleared eight at a time)
    alignas(8) uint8_t low[C::NP];    // 1: lowered by this run, at C::mine(); 2: a source on its first run
};

template <int TX, int TY, int TZ, int OP = 0, bool COUNT = false>
__global__ void __launch_bounds__((64 * SweepCfg<TX, TY, TZ>::W))
    __attribute__((amdgpu_waves_per_eu((SweepCfg<TX, TY, TZ>::WPE)))) k_sweep(SolveArgs A) {
    using C = SweepCfg<TX, TY, TZ>;
    using F = Face<TX, TY, TZ>;
    static_assert(OP == 0 || OP == 4, "the monotone operators");
    constexpr int NPT = C::NPT;
    __shared__ SweepTile<TX, TY, TZ, OP> s_tiles[C::W];
    __shared__ GroupMail s_mail;
    if (threadIdx.x == 0) {
        s_mail.lock = 0;
        s_mail.idle = 0;
    }
    __syncthreads();  // the waves part here; none meets another one again

    const int w = uni((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    double* const sT = s_tiles[w].t;
    double* const sQ = s_tiles[w].q;
    double* const sW = s_tiles[w].wx;
    uint8_t* const sF = s_tiles[w].dirty;
    uint8_t* const sC = s_tiles[w].low;
    unsigned long long* const s_stat = s_tiles[w].stat;
    const Sched& S = A.s;
    // this lane's column in sweep order (y and z counted from the side the sweep starts at)
    const int yy = lane % TY, zz = (lane / TY) % TZ;
    const int xs0 = ((lane / C::NCOL) * NPT - yy - zz) & (TX - 1);  // its first point of a sweep
    // lanes with a neighbour column ahead and behind along y and z
    constexpr unsigned long long aheadY = C::inner(1, 1), behindY = C::inner(1, 0);
    constexpr unsigned long long aheadZ = C::inner(2, 1), behindZ = C::inner(2, 0);
    unsigned long long w_eval = 0, w_imp = 0, w_good = 0;
    if (lane == 0) {
        for (int i = 0; i < 8; ++i) s_stat[i] = 0;
        s_stat[8] = wall_clock64();
    }
    int32_t cur_hint = 0;
    int64_t slot = 0;
    int next = -1;
    for (;;) {
        // ---- claim (or take the tile handed on) ----------------------------
        int tile = next;
        if (tile < 0) tile = claim_group(S, s_mail, w, &slot, cur_hint);
        else if (lane == 0) ++s_stat[7];
        tile = uni(tile);
        if (tile < 0) break;
        uint32_t st = 0;
        if (lane == 0) {
            st = __hip_atomic_fetch_xor(S.tstate + tile, kQ | kR, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((st & (kQ | kR)) != kQ) set_flag(S, kFlagWatchdog);
            if (S.max_visits > 0) {
                unsigned long long v = __hip_atomic_fetch_add(S.counters + 3, 1ull, __ATOMIC_RELAXED,
                                                              __HIP_MEMORY_SCOPE_AGENT);
                if ((long long)v >= S.max_visits) {
                    set_flag(S, kFlagLimit);
                    st |= 0x80000000u;  // skip marker
                }
            }
            ++s_stat[4];
            const unsigned long long now = wall_clock64();
            s_stat[0] += now - s_stat[8];
            s_stat[8] = now;
        }
        st = (uint32_t)uni((int)st);
        stores_done();  // the RMW has returned: every load of this run comes after it
        next = -1;
        if (st & 0x80000000u) {  // visit cap reached: drop the tile
            if (lane == 0) drop_run(S, (uint32_t)tile, slot);
            continue;
        }
        const bool visited = (st & kV) != 0;
        const Prob P = wave_prob_of_tile(A.pt, tile);
        const int tl = tile - P.tile_off;
        const int tx = tl % P.ntx, ty = (tl / P.ntx) % P.nty, tz = tl / (P.ntx * P.nty);
        const int x0 = tx * TX, y0 = ty * TY, z0 = tz * TZ;
        // Optional bucket horizon (k = S.horizon > 0): a run settles only values
        // with floor(r / delta) < b + k, b its bucket (with k = 1 the bucket
        // discipline of delta-stepping).  A lower value never depends on a
        // higher one (the operator is causal), so nothing below the horizon is
        // lost; larger candidates are left for a later run of this tile, keyed
        // by the smallest of them.
        const double hz = (double)(slot_bucket(slot) + S.horizon);

        // ---- stage the tile and its halo in LDS ----------------------------
        // every load goes out before any is used: one memory round trip
        constexpr int HB[6] = {(F::cells(0) + 63) / 64, (F::cells(1) + 63) / 64, (F::cells(2) + 63) / 64,
                               (F::cells(3) + 63) / 64, (F::cells(4) + 63) / 64, (F::cells(5) + 63) / 64};
        constexpr int HPT = 2 * (HB[0] + HB[2] + (C::D3 ? HB[4] : 0));  // halo loads per lane
        const int64_t plane = (int64_t)P.ny * P.nx;
        const int64_t g0 = P.pt_off + z0 * plane + (int64_t)y0 * P.nx + x0;  // the tile's first point
        // which faces have a neighbour tile (bit f)
        const int has = (tx > 0 ? 1 : 0) | (tx < P.ntx - 1 ? 2 : 0) | (ty > 0 ? 4 : 0) | (ty < P.nty - 1 ? 8 : 0) |
                        (tz > 0 ? 16 : 0) | (tz < P.ntz - 1 ? 32 : 0);
        // this lane's first point, and whether it and the tile's rows are in the grid
        const int lx0 = lane % TX, ly0 = (lane / TX) % TY, lz0 = lane / (TX * TY);
        const int nx = P.nx - x0, ny = P.ny - y0, nz = P.nz - z0;  // points from the tile's first on
        const bool whole = nx >= TX && ny >= TY && nz >= TZ;
        const bool narrow = offsets_fit_32<TX, TY, TZ>(P.nx, plane);
        const int64_t lane_off = lz0 * plane + (int64_t)ly0 * P.nx + lx0;
        {
            double fv[NPT], tv[NPT], hv[HPT];
            if (whole && narrow) {
                // Tiles wholly inside the grid: no bounds checks, and 32-bit byte
                // offsets from the corner of the halo, common to t and the field.
                const int64_t corner = g0 - (C::D3 ? plane : 0) - P.nx - 1;
                const char* const tb = (const char*)(A.t + corner);
                const char* const fb = (const char*)(A.field + corner);
                const uint32_t row = 8u * (uint32_t)P.nx, pln = 8u * (uint32_t)plane;
                auto off = [&](int lx, int ly, int lz) {
                    return (C::D3 ? (uint32_t)(lz + 1) * pln : 0u) + (uint32_t)(ly + 1) * row + 8u * (uint32_t)(lx + 1);
                };
                auto ld = [&](uint32_t o) {
                    return as_f64(__hip_atomic_load((const uint64_t*)(tb + o), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                };
                const uint32_t o0 = off(lx0, ly0, lz0);
#pragma unroll
                for (int j = 0; j < NPT; ++j) {
                    const uint32_t o = o0 + ((uint32_t)C::jz(j) * pln + (uint32_t)C::jy(j) * row + 8u * (uint32_t)C::jx(j));
                    fv[j] = *(const double*)(fb + o);
                    tv[j] = ld(o);
                }
                int hk = 0;
#pragma unroll
                for (int f = 0; f < C::NF; ++f) {
#pragma unroll
                    for (int b = 0; b < HB[f]; ++b, ++hk) {
                        const int c = lane + b * 64;
                        hv[hk] = inf64();
                        if (((has >> f) & 1) == 0) continue;
                        if (F::cells(f) % 64 != 0 && c >= F::cells(f)) continue;
                        const F e(f, c);
                        const int s = (f & 1) ? 1 : -1;
                        hv[hk] = ld(off(e.lx + (f < 2 ? s : 0), e.ly + (f >> 1 == 1 ? s : 0), e.lz + (f >= 4 ? s : 0)));
                    }
                }
            } else {
#pragma unroll
                for (int j = 0; j < NPT; ++j) {
                    const int64_t step = g0 + C::jz(j) * plane + (int64_t)C::jy(j) * P.nx + C::jx(j);
                    fv[j] = 1.0;
                    tv[j] = inf64();
                    if (!(lx0 + C::jx(j) < nx && ly0 + C::jy(j) < ny && lz0 + C::jz(j) < nz)) continue;
                    fv[j] = (A.field + step)[lane_off];
                    tv[j] = as_f64(__hip_atomic_load((const uint64_t*)(A.t + step) + lane_off, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT));
                }
                int hk = 0;
#pragma unroll
                for (int f = 0; f < C::NF; ++f) {
#pragma unroll
                    for (int b = 0; b < HB[f]; ++b, ++hk) {
                        const int c = lane + b * 64;
                        hv[hk] = inf64();
                        if (((has >> f) & 1) == 0) continue;
                        if (F::cells(f) % 64 != 0 && c >= F::cells(f)) continue;
                        const F e(f, c);
                        if (!(e.lx < nx && e.ly < ny && e.lz < nz)) continue;
                        const int64_t step = f < 2 ? 1 : (f < 4 ? (int64_t)P.nx : plane);
                        const double* from = A.t + (g0 + ((f & 1) ? step : -step));
                        hv[hk] = as_f64(__hip_atomic_load((const uint64_t*)from + (e.lz * plane + (int64_t)e.ly * P.nx + e.lx),
                                                          __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                    }
                }
            }
            if constexpr (OP == 4) {
                // clamped past the grid's end, where no point is relaxed
                constexpr int NW = 2 * (TX + TY + TZ);
                for (int i = lane; i < NW; i += 64) {
                    int k = i, n = TX, off = 0, o = x0, m = P.nx;
                    if (k >= 2 * TX) {
                        k -= 2 * TX;
                        n = TY, off = 2 * P.nx, o = y0, m = P.ny;
                        if (k >= 2 * TY) {
                            k -= 2 * TY;
                            n = TZ, off = 2 * (P.nx + P.ny), o = z0, m = P.nz;
                        }
                    }
                    const int side = k >= n ? 1 : 0;
                    sW[i] = A.rw[off + side * m + min(o + k - side * n, m - 1)];
                }
            }
            for (int i = lane; i < C::NP / 8; i += 64) {
                ((uint64_t*)sF)[i] = 0;
                ((uint64_t*)sC)[i] = 0;
            }
            unsigned long long bad = 0;
#pragma unroll
            for (int j = 0; j < NPT; ++j) {
                bool ok;
                double q = field_q(fv[j], P.h, P.kind, ok);
                bad |= __ballot(!ok);
                // a source (sign bit) is never relaxed
                q = signbit(tv[j]) ? 0.0 : q;
                sT[C::lds(lx0 + C::jx(j), ly0 + C::jy(j), lz0 + C::jz(j))] = fabs(tv[j]);
                sQ[lane + j * 64] = q;
            }
            if (bad || !whole) {
                // nor is a point outside the grid or the field's domain
#pragma unroll
                for (int j = 0; j < NPT; ++j) {
                    const bool in = lx0 + C::jx(j) < nx && ly0 + C::jy(j) < ny && lz0 + C::jz(j) < nz;
                    bool ok;
                    (void)field_q(fv[j], P.h, P.kind, ok);
                    if (in && !ok) set_flag(S, kFlagDomain);
                    if (!in || !ok) sQ[lane + j * 64] = 0.0;
                }
            }
            wave_order();
            // First marks.  A point can improve only next to a smaller value.
            // The interior is at the fixed point its last run left given the
            // old halo, or +inf before a first run, so only points next to a
            // smaller halo value count, except in a tile holding a source, on
            // a warm start's first run and with a horizon (points left beyond
            // it last time), where every neighbour counts.
            int hk = 0;
#pragma unroll
            for (int f = 0; f < C::NF; ++f) {
#pragma unroll
                for (int b = 0; b < HB[f]; ++b, ++hk) {
                    const int c = lane + b * 64;
                    if (F::cells(f) % 64 == 0 || c < F::cells(f)) {
                        const F e(f, c);
                        const int L = e.lds();
                        const double h = fabs(hv[hk]);
                        sT[L + F::out(f)] = h;
                        if (h < sT[L]) sF[e.point()] = 1;
                    }
                }
            }
            wave_order();
        }
        if ((st & kS) || S.horizon > 0 || (!visited && A.warm)) {
#pragma unroll 1
            for (int j = 0; j < NPT; ++j) {
                const int p = lane + j * 64;
                const int L = C::lds(p % TX, (p / TX) % TY, p / (TX * TY));
                double m = nmin(nmin(sT[L - 1], sT[L + 1]), nmin(sT[L - C::SY], sT[L + C::SY]));
                if (C::D3) m = nmin(m, nmin(sT[L - C::SZ], sT[L + C::SZ]));
                if (m < sT[L]) sF[p] = 1;
                // The first run hands a source's value to the neighbours across
                // the faces (2: its own value is not stored): it is not lowered,
                // and in a tile of one point nothing else is.
                if ((st & kS) && !visited && !(sQ[p] > 0.0) && sT[L] < inf64()) sC[C::mine(p)] = 2;
            }
        }
        // The octant to sweep first: per axis, the side where more of the
        // halo (up to 64 cells a face) is the smaller one.
        int mx, my, mz = 0;
        {
            constexpr int NX = TY * TZ, NY = TX * TZ, NZ = TX * TY;
            int c = NX >= 64 ? lane * (NX / 64) : lane % NX;
            double a = sT[C::lds(-1, c % TY, c / TY)], b = sT[C::lds(TX, c % TY, c / TY)];
            mx = __popcll(__ballot(a < b)) >= __popcll(__ballot(b < a)) ? 0 : TX - 1;
            c = NY >= 64 ? lane * (NY / 64) : lane % NY;
            a = sT[C::lds(c % TX, -1, c / TX)];
            b = sT[C::lds(c % TX, TY, c / TX)];
            my = __popcll(__ballot(a < b)) >= __popcll(__ballot(b < a)) ? 0 : TY - 1;
            if (C::D3) {
                c = NZ >= 64 ? lane * (NZ / 64) : lane % NZ;
                a = sT[C::lds(c % TX, c / TX, -1)];
                b = sT[C::lds(c % TX, c / TX, TZ)];
                mz = __popcll(__ballot(a < b)) >= __popcll(__ballot(b < a)) ? 0 : TZ - 1;
            }
        }
        wave_order();
        if (lane == 0) {
            const unsigned long long now = wall_clock64();
            s_stat[1] += now - s_stat[8];
            s_stat[8] = now;
        }

        // ---- relax until the tile is quiet --------------------------------
        double pend = inf64();
        int passes = 0;  // levels with work
        {
            const bool held = S.horizon > 0;
            int sweeps = 0;
            bool turn = true;
            uint32_t D = 0;
            int xs = 0, base = 0, pc = 0, cy = 0, cz = 0;
            int ax = 0, ay = 0, az = 0;  // LDS steps ahead along each axis
            for (;;) {
                if (turn) {
                    // this lane's column and dirty bits under the octant
                    cy = yy ^ my;
                    cz = zz ^ mz;
                    base = C::lds(0, cy, cz);
                    pc = (cz * TY + cy) * TX;
                    xs = xs0;
                    ax = mx ? -1 : 1;
                    ay = my ? -C::SY : C::SY;
                    az = mz ? -C::SZ : C::SZ;
                    D = 0;
                    wave_order();
#pragma unroll
                    for (int j = 0; j < NPT; ++j) D |= (uint32_t)sF[pc + (((xs0 + j) & (TX - 1)) ^ mx)] << j;
                    wave_order();
                    for (int i = lane; i < C::NP / 8; i += 64) ((uint64_t*)sF)[i] = 0;
                }
                bool quiet = false;
                for (int k = 0; k < C::SPAN; ++k) {
                    unsigned long long act = __ballot(D & 1u);
                    if (!act) {
                        quiet = !__ballot(D != 0u);
                        if (quiet) break;
                        do {  // levels without a dirty point
                            D >>= 1;
                            ++xs;
                            ++k;
                            act = __ballot(D & 1u);
                        } while (!act);
                        xs &= TX - 1;
                    }
                    wave_order();
                    const int x = xs ^ mx;
                    double* const pt = sT + base + x;
                    const double q = sQ[pc + x];
                    const double tc = pt[0];
                    const double xa = pt[ax], xb = pt[-ax], ya = pt[ay], yb = pt[-ay];
                    const double za = C::D3 ? pt[az] : inf64(), zb = C::D3 ? pt[-az] : inf64();
                    act &= mask_lt(0.0, q);
                    ++passes;
                    double r;
                    if constexpr (OP == 0) {
                        r = update_short<C::D3>(nmin(xa, xb), nmin(ya, yb), nmin(za, zb), q, tc, act);
                    } else {
                        // behind and ahead along each axis: the operator does not
                        // tell an axis's two sides apart
                        const double nb6[6] = {xb, xa, yb, ya, zb, za};
                        const int ox = mx ? TX : 0, oy = 2 * TX + (my ? TY : 0), oz = 2 * (TX + TY) + (mz ? TZ : 0);
                        const double w6[6] = {sW[ox + x], sW[(TX - ox) + x], sW[oy + cy], sW[(4 * TX + TY - oy) + cy],
                                              C::D3 ? sW[oz + cz] : 1.0,
                                              C::D3 ? sW[(4 * (TX + TY) + TZ - oz) + cz] : 1.0};
                        r = update_rect_short<C::D3>(nb6, w6, q, tc, act);
                    }
                    unsigned long long chm = mask_lt(r, tc) & act;
                    if (held) {
                        // values at or beyond bucket hz are held back; one whose bucket
                        // index overflows the range is settled at once, so the requeue
                        // can never repeat forever
                        const double rb = r * S.inv_delta;
                        const unsigned long long keep = chm & mask_ge(rb, hz) & mask_lt(rb, 1.0e15);
                        if (in_mask(keep)) pend = nmin(pend, r);
                        chm &= ~keep;
                    }
                    if (in_mask(chm)) {
                        pt[0] = r;
                        sC[C::mine(pc + x)] = 1;
                    }
                    // neighbours above the new value may improve (the operator is causal)
                    const double rl = in_mask(chm) ? r : inf64();
                    unsigned long long a = mask_lt(rl, xa) & __ballot(xs < TX - 1);
                    unsigned long long b = mask_lt(rl, xb) & __ballot(xs > 0);
                    a |= (mask_lt(rl, ya) & aheadY) << 1;
                    b |= (mask_lt(rl, yb) & behindY) >> 1;
                    if (C::D3) {
                        // in a full wave of columns the last plane's bits leave at the end
                        a |= (mask_lt(rl, za) & (C::NCOL < 64 ? aheadZ : ~0ull)) << TY;
                        b |= (mask_lt(rl, zb) & (C::NCOL < 64 ? behindZ : ~0ull)) >> TY;
                    }
                    // a point behind is next visited by the lane one place back along its column
                    if constexpr (C::NCOL < 64) b = (b >> C::NCOL) | (b << (64 - C::NCOL));
                    D = (D >> 1) | (in_mask(a) ? 1u : 0u) | (in_mask(b) ? 1u << (NPT - 2) : 0u);
                    xs = (xs + 1) & (TX - 1);
                    if constexpr (COUNT) {
                        bool good = false;
                        if (in_mask(chm)) {
                            const int gx = x0 + x, gy = y0 + cy, gz = z0 + cz;
                            good = r == A.work_ref[P.pt_off + ((int64_t)gz * P.ny + gy) * P.nx + gx];
                        }
                        w_eval += __popcll(act);
                        w_imp += __popcll(chm);
                        w_good += __popcll(__ballot(good));
                    }
                }
                if (quiet) break;
                if (++sweeps > (1 << 20)) {
                    if (lane == 0) set_flag(S, kFlagWatchdog);
                    break;
                }
                // The next sweep turns round along the axes where most lanes' next
                // dirty point has its smaller neighbour ahead; the dirty bits then go
                // through LDS to the lanes that visit those points.
                int tx2 = 0, ty2 = 0, tz2 = 0;
                {
                    wave_order();
                    const bool any = D != 0u;
                    const double* const pt = sT + base + (((xs + (any ? __ffs((int)D) - 1 : 0)) & (TX - 1)) ^ mx);
                    const double xa = pt[ax], xb = pt[-ax], ya = pt[ay], yb = pt[-ay];
                    if (__popcll(__ballot(any && xa < xb)) > __popcll(__ballot(any && xb < xa))) tx2 = TX - 1;
                    if (__popcll(__ballot(any && ya < yb)) > __popcll(__ballot(any && yb < ya))) ty2 = TY - 1;
                    if (C::D3) {
                        const double za = pt[az], zb = pt[-az];
                        if (__popcll(__ballot(any && za < zb)) > __popcll(__ballot(any && zb < za))) tz2 = TZ - 1;
                    }
                }
                turn = (tx2 | ty2 | tz2) != 0;
                if (turn) {
                    wave_order();
#pragma unroll
                    for (int j = 0; j < NPT; ++j)
                        if ((D >> j) & 1u) sF[pc + (((xs + j) & (TX - 1)) ^ mx)] = 1;
                    mx ^= tx2;
                    my ^= ty2;
                    mz ^= tz2;
                }
            }
        }
        wave_order();
        if (lane == 0) {
            const unsigned long long now = wall_clock64();
            s_stat[2] += now - s_stat[8];
            s_stat[8] = now;
        }

        // ---- write back lowered points, gather lowered face minima ---------
        int upd = 0;
#pragma unroll
        for (int j = 0; j < NPT; ++j) {
            const bool c = sC[lane * NPT + j] == 1;  // only points in the grid are ever lowered
            const unsigned long long m = __ballot(c);
            if (m) {
                const int64_t step = g0 + C::jz(j) * plane + (int64_t)C::jy(j) * P.nx + C::jx(j);
                if (c) tstore(A.t + step + lane_off, sT[C::lds(lx0 + C::jx(j), ly0 + C::jy(j), lz0 + C::jz(j))]);
                upd += __popcll(m);
            }
        }
        // A lowered face value matters to the neighbour only where it is below
        // the neighbour's own value there (its halo cell here, as staged).  Lane f
        // gets face f's key.
        unsigned long long face = kInfBits;
#pragma unroll
        for (int f = 0; f < C::NF; ++f) {
            if (!((has >> f) & 1)) continue;
            double fk = inf64();
            unsigned long long any = 0;
#pragma unroll
            for (int b = 0; b < HB[f]; ++b) {
                const int c = lane + b * 64;
                const bool in = F::cells(f) % 64 == 0 || c < F::cells(f);
                const F e(f, in ? c : 0);
                const int L = e.lds();
                const double v = sT[L];
                const bool low = in && sC[C::mine(e.point())] != 0 && v < sT[L + F::out(f)];
                fk = low ? nmin(fk, v) : fk;
                any |= __ballot(low);
            }
            if (any) {
                const uint64_t m = wave_min_u64(as_u64(fk));
                if (lane == f) face = m;
            }
        }
        unsigned long long self_key = kInfBits;
        if (__ballot(pend < inf64())) self_key = as_u64(wave_min(pend));
        // face neighbours x-, x+, y-, y+, z-, z+ (bit 30: the tile exists)
        uint32_t nb = 0, nid = 0;
        if (lane < 6) {
            const int d = lane >> 1;
            const int step = d == 0 ? 1 : (d == 1 ? P.ntx : P.ntx * P.nty);
            if ((has >> lane) & 1) {
                nid = (uint32_t)(tile + ((lane & 1) ? step : -step));
                nb = 0x40000000u;
            }
        }
        // the stores complete before the tile's faces are handed to the neighbours
        stores_done();
        next = uni(publish_wave(S, A.tkey, (uint32_t)tile, slot, !visited, nb, nid, face, true, self_key));
        if (lane == 0) {
            s_stat[5] += (unsigned long long)upd;
            s_stat[6] += (unsigned long long)passes;
            const unsigned long long now = wall_clock64();
            s_stat[3] += now - s_stat[8];
            s_stat[8] = now;
        }
    }
    if (COUNT && lane == 0) {
        __hip_atomic_fetch_add(S.counters + 16, w_eval, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(S.counters + 17, w_imp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(S.counters + 18, w_good, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (lane == 0) {
        s_stat[0] += wall_clock64() - s_stat[8];
        flush_stats(S, s_stat);
    }
}

}  // namespace eik
