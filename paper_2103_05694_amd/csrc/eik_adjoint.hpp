// Adjoint (reverse) sweep: gradient of a travel-time loss with respect to
// slowness through the recorded upwind dependency graph.
//
// The paper gives no gradient; it is the implicit derivative of the discrete
// equations of Eq. (difference_as_root) -- sum over upwind axes of
// (t_n - t_{p_k})^2 = q_n^2 with q_n = h * s_n -- over the upwind parents p_k
// the forward pass recorded.  Writing w_{n,k} = fl(t_n - t_{p_k}) and
// W_n = fl(fl(w_x + w_y) + w_z):
//   lambda_n = g_n + sum over children m (n is m's axis-k parent) of
//              fl(mu_m * w_{m,k}), summed in neighbour order x-,x+,y-,y+,z-,z+,
//   mu_n     = fl(lambda_n / W_n),
//   dL/ds_n  = fl(fl(mu_n * q_n) * h),  sources: 0
// (the last line in a separate elementwise pass, k_adj_grad, once every mu is
// final: the sweep itself never reads the field).
// A child always has a strictly larger time than its parent, so the graph is
// acyclic and mu can be evaluated children-first.
//
// The sweep reuses the forward scheduler with tiles as work items, but is
// readiness-driven: a point is evaluated exactly once, when every child (in the
// tile or in the halo) is done, so each mu is a fixed function of final values
// and the result is deterministic whatever the visit order.  "Not done" is a
// NaN in mu, which is filled with NaN before the sweep; a point's mu goes from
// NaN to its final value once, so any read returns one or the other.  Tiles are
// prioritised by decreasing time (key tref - t), and a finished face point
// activates the neighbour tile holding its parent.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "eik_sweep.hpp"

namespace eik {

__device__ __forceinline__ double qnan64() { return as_f64(0x7FF8000000000000ull); }

// Before the sweep, in one pass: mu := NaN ("not done") everywhere, so a point
// of a tile that has not run yet reads as not done without looking at the
// tile's state; per tile the largest time (key source); and the launch's
// largest time.  A wave per tile; the launch-wide maximum leaves a block once
// and only where it is larger than what is there (an atomic per tile on that
// one word took 3.2 ms for 262144 tiles, against 0.9 ms to move t and mu).
template <int TX, int TY, int TZ>
__global__ void __launch_bounds__(256) k_adj_prep(ProbTable T, int ntiles, const double* t, double* mu,
                                                  uint64_t* tile_tmax, unsigned long long* tref_bits) {
    __shared__ unsigned long long s_m;
    if (threadIdx.x == 0) s_m = 0ull;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    unsigned long long largest = 0ull;
    for (int tile = uni((int)(blockIdx.x * 4 + (threadIdx.x >> 6))); tile < ntiles; tile += (int)gridDim.x * 4) {
        const Prob P = wave_prob_of_tile(T, tile);
        const int tl = tile - P.tile_off;
        const int tx = tl % P.ntx, ty = (tl / P.ntx) % P.nty, tz = tl / (P.ntx * P.nty);
        unsigned long long m = 0ull;
#pragma unroll
        for (int j = 0; j < TX * TY * TZ / 64; ++j) {
            const int i = lane + j * 64;
            const int x = tx * TX + i % TX, y = ty * TY + (i / TX) % TY, z = tz * TZ + i / (TX * TY);
            if (x < P.nx && y < P.ny && z < P.nz) {
                const int64_t gi = P.pt_off + ((int64_t)z * P.ny + y) * P.nx + x;
                const double v = fabs(t[gi]);
                mu[gi] = qnan64();
                if (v < inf64() && as_u64(v) > m) m = as_u64(v);
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const unsigned long long o = __shfl_xor(m, off);
            m = o > m ? o : m;
        }
        if (lane == 0) tile_tmax[tile] = m;
        largest = m > largest ? m : largest;
    }
    if (lane == 0) atomicMax(&s_m, largest);
    __syncthreads();
    if (threadIdx.x == 0 && s_m > __hip_atomic_load(tref_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        __hip_atomic_fetch_max(tref_bits, s_m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Queue every tile, latest first.  Lanes that push into the same ring do so
// with one read-modify-write per counter for all of them (a counter's line
// takes one about every 12 ns, and there are as many tiles as points / 1024).
__global__ void k_adj_push_all(int ntiles, const uint64_t* tile_tmax,
                               const unsigned long long* tref_bits, Sched s) {
    const double tref = as_f64(*tref_bits);
    const int lane = threadIdx.x & 63;
    if (blockIdx.x == 0 && threadIdx.x == 0) *s.poisoned = 0;  // rings were wiped by the reset
    for (int first = blockIdx.x * blockDim.x + (threadIdx.x & ~63); first < ntiles; first += gridDim.x * blockDim.x) {
        const int tile = first + lane;
        const bool in = tile < ntiles;
        if (in) s.tstate[tile] = kQ;
        const int64_t k = in ? push_bucket(s, tref - as_f64(tile_tmax[tile]), 0, 0) : 0;
        const int r = ring_of(k, shard_of((uint32_t)tile));
        unsigned long long todo = __ballot(in);
        if (lane == 0) pend_add(s, (uint32_t)__popcll(todo), 0);
        while (todo) {
            const int lead = __ffsll((long long)todo) - 1;
            const int ring = __shfl(r, lead);
            const unsigned long long same = __ballot(r == ring) & todo;
            todo &= ~same;
            uint32_t pos = 0;
            if (lane == lead)
                pos = __hip_atomic_fetch_add(ring_tail(s, ring), (uint32_t)__popcll(same), __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
            pos = __shfl(pos, lead) + (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
            if ((same >> lane) & 1ull) {
                // nothing runs yet: every cell of an empty ring is free
                uint64_t* cell = s.items + (size_t)ring * (s.cap_mask + 1) + (pos & s.cap_mask);
                __hip_atomic_store(cell, ((uint64_t)(pos + 1u) << 32) | (uint32_t)tile, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
            if (lane == lead) cr_add(s, ring, (uint64_t)__popcll(same));
        }
    }
}

// dL/ds from the final multipliers: fl(fl(mu * q) * h) at non-sources, 0 at
// sources (mu is 0 there); a field value outside the domain raises the flag.
// One block per tile, so that a tile's rows are read and written together.
template <int TX, int TY, int TZ>
__global__ void k_adj_grad(ProbTable T, int ntiles, const double* field, const uint8_t* par, const double* mu,
                           double* grad, uint32_t* flags) {
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const Prob P = prob_of_tile(T, tile);
        const int tl = tile - P.tile_off;
        const int tx = tl % P.ntx, ty = (tl / P.ntx) % P.nty, tz = tl / (P.ntx * P.nty);
        for (int i = threadIdx.x; i < TX * TY * TZ; i += blockDim.x) {
            const int x = tx * TX + i % TX, y = ty * TY + (i / TX) % TY, z = tz * TZ + i / (TX * TY);
            if (!(x < P.nx && y < P.ny && z < P.nz)) continue;
            const int64_t gi = P.pt_off + ((int64_t)z * P.ny + y) * P.nx + x;
            bool ok;
            const double q = field_q(field[gi], P.h, P.kind, ok);
            if (!ok) __hip_atomic_fetch_or(flags, kFlagDomain, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            grad[gi] = (par[gi] & 0x80) ? 0.0 : (mu[gi] * (ok ? q : 0.0)) * P.h;
        }
    }
}

struct AdjArgs {
    ProbTable pt;
    const double* t;
    const uint8_t* par;
    const double* g;
    double* mu;
    uint64_t* tkey;
    const unsigned long long* tref_bits;
    Sched s;
};

// One wave's tile of the adjoint in LDS.
template <int TX, int TY, int TZ>
struct AdjTile {
    using C = SweepCfg<TX, TY, TZ>;
    double t[C::NLDS];
    double m[C::NLDS];            // mu of a finished point, dL/dt of one that is not (halo: mu)
    unsigned long long stat[9];   // as in Block
    alignas(8) uint8_t dirty[C::NP];  // marks carried into the next sweep (cleared eight at a time)
    uint8_t par[C::NLDS];         // parent codes (bits 0-5), kDone, 0x80 a source or outside the grid
};
constexpr uint32_t kDone = 0x40u;

// Waves (tiles in flight) per workgroup: as many as a compute unit's LDS holds.
template <int TX, int TY, int TZ>
constexpr int adj_waves() {
    return (160 * 1024 - 1024) / (int)sizeof(AdjTile<TX, TY, TZ>) < 16
               ? (160 * 1024 - 1024) / (int)sizeof(AdjTile<TX, TY, TZ>)
               : 16;
}

// The reverse sweep, one wave per tile in the order of the forward solver
// (eik_sweep.hpp) turned round: the octant is the one the parents lie in, so a
// point is mostly visited after its children, and a point that finishes marks
// its parents, which are then mostly the next points visited.  Most levels only
// look up readiness; the FP64 part runs when some lane's point is ready.
//
// Bound by the chain of tiles from the last points reached back to the source
// (a level 0.45 us, a run 22 us, of which staging and publishing 10), and with
// many problems by latency at 5 tiles of 16x8x8 in flight a compute unit.  A
// workgroup per tile with a barrier per readiness pass took 53.5 ms for 32
// problems of 256x256x128 (16x8x8 tiles), this takes 31.7 ms.
template <int TX, int TY, int TZ>
__global__ void __launch_bounds__((64 * adj_waves<TX, TY, TZ>()))
    __attribute__((amdgpu_waves_per_eu(((adj_waves<TX, TY, TZ>() + 3) / 4)))) k_adjoint(AdjArgs A) {
    using C = SweepCfg<TX, TY, TZ>;
    using F = Face<TX, TY, TZ>;
    constexpr int NPT = C::NPT;
    __shared__ AdjTile<TX, TY, TZ> s_tiles[adj_waves<TX, TY, TZ>()];
    __shared__ GroupMail s_mail;
    if (threadIdx.x == 0) {
        s_mail.lock = 0;
        s_mail.idle = 0;
    }
    __syncthreads();  // the waves part here; none meets another one again

    const int w = uni((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    double* const sT = s_tiles[w].t;
    double* const sM = s_tiles[w].m;
    uint8_t* const sP = s_tiles[w].par;
    uint8_t* const sF = s_tiles[w].dirty;
    unsigned long long* const s_stat = s_tiles[w].stat;
    const Sched& S = A.s;
    const double tref = as_f64(*A.tref_bits);
    // this lane's column in sweep order (y and z counted from the side the sweep starts at)
    const int yy = lane % TY, zz = (lane / TY) % TZ;
    const int xs0 = ((lane / C::NCOL) * NPT - yy - zz) & (TX - 1);  // its first point of a sweep
    constexpr unsigned long long aheadY = C::inner(1, 1), behindY = C::inner(1, 0);
    constexpr unsigned long long aheadZ = C::inner(2, 1), behindZ = C::inner(2, 0);
    if (lane == 0) {
        for (int i = 0; i < 8; ++i) s_stat[i] = 0;
        s_stat[8] = wall_clock64();
    }
    auto phase = [&](int i) {
        if (lane == 0) {
            const unsigned long long now = wall_clock64();
            s_stat[i] += now - s_stat[8];
            s_stat[8] = now;
        }
    };
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
            ++s_stat[4];
        }
        st = (uint32_t)uni((int)st);
        phase(0);
        stores_done();  // the RMW has returned: every load of this run comes after it
        next = -1;
        const bool visited = (st & kV) != 0;
        const Prob P = wave_prob_of_tile(A.pt, tile);
        const int tl = tile - P.tile_off;
        const int tx = tl % P.ntx, ty = (tl / P.ntx) % P.nty, tz = tl / (P.ntx * P.nty);
        const int x0 = tx * TX, y0 = ty * TY, z0 = tz * TZ;

        // ---- stage the tile and its halo: every load goes out before any is used
        constexpr int HB[6] = {(F::cells(0) + 63) / 64, (F::cells(1) + 63) / 64, (F::cells(2) + 63) / 64,
                               (F::cells(3) + 63) / 64, (F::cells(4) + 63) / 64, (F::cells(5) + 63) / 64};
        constexpr int HPT = 2 * (HB[0] + HB[2] + (C::D3 ? HB[4] : 0));  // halo cells per lane
        const int64_t plane = (int64_t)P.ny * P.nx;
        const int64_t g0 = P.pt_off + z0 * plane + (int64_t)y0 * P.nx + x0;  // the tile's first point
        const int has = (tx > 0 ? 1 : 0) | (tx < P.ntx - 1 ? 2 : 0) | (ty > 0 ? 4 : 0) | (ty < P.nty - 1 ? 8 : 0) |
                        (tz > 0 ? 16 : 0) | (tz < P.ntz - 1 ? 32 : 0);
        const int lx0 = lane % TX, ly0 = (lane / TX) % TY, lz0 = lane / (TX * TY);
        const int nx = P.nx - x0, ny = P.ny - y0, nz = P.nz - z0;  // points from the tile's first on
        const bool whole = nx >= TX && ny >= TY && nz >= TZ;
        const bool narrow = offsets_fit_32<TX, TY, TZ>(P.nx, plane);
        const int64_t lane_off = lz0 * plane + (int64_t)ly0 * P.nx + lx0;
        uint32_t was = 0;  // bit j: point lane + 64 j was finished (or is outside) when the run began
        {
            double tv[NPT], gv[NPT], mv[NPT], ht[HPT], hm[HPT];
            uint8_t pv[NPT], hp[HPT];
            if (whole && narrow) {
                // no bounds checks, 32-bit offsets from the corner of the halo
                const int64_t corner = g0 - (C::D3 ? plane : 0) - P.nx - 1;
                const double* const tb = A.t + corner;
                const double* const gb = A.g + corner;
                const double* const mb = A.mu + corner;
                const uint8_t* const pb = A.par + corner;
                const uint32_t row = (uint32_t)P.nx, pln = (uint32_t)plane;
                auto off = [&](int lx, int ly, int lz) {
                    return (C::D3 ? (uint32_t)(lz + 1) * pln : 0u) + (uint32_t)(ly + 1) * row + (uint32_t)(lx + 1);
                };
                auto ld = [&](const double* b, uint32_t o) { return *(const double*)((const char*)b + 8u * o); };
                auto ldm = [&](uint32_t o) {
                    return as_f64(__hip_atomic_load((const uint64_t*)((const char*)mb + 8u * o), __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT));
                };
                const uint32_t o0 = off(lx0, ly0, lz0);
#pragma unroll
                for (int j = 0; j < NPT; ++j) {
                    const uint32_t o = o0 + ((uint32_t)C::jz(j) * pln + (uint32_t)C::jy(j) * row + (uint32_t)C::jx(j));
                    pv[j] = pb[o];
                    tv[j] = ld(tb, o);
                    gv[j] = ld(gb, o);
                    mv[j] = ldm(o);
                }
                int hk = 0;
#pragma unroll
                for (int f = 0; f < C::NF; ++f) {
#pragma unroll
                    for (int b = 0; b < HB[f]; ++b, ++hk) {
                        const int c = lane + b * 64;
                        ht[hk] = inf64();
                        hm[hk] = 0.0;
                        hp[hk] = 0x80;  // outside cells act as finished sources
                        if (((has >> f) & 1) == 0) continue;
                        if (F::cells(f) % 64 != 0 && c >= F::cells(f)) continue;
                        const F e(f, c);
                        const int s = (f & 1) ? 1 : -1;
                        const uint32_t o = off(e.lx + (f < 2 ? s : 0), e.ly + (f >> 1 == 1 ? s : 0), e.lz + (f >= 4 ? s : 0));
                        hp[hk] = pb[o];
                        ht[hk] = ld(tb, o);
                        hm[hk] = ldm(o);
                    }
                }
            } else {
#pragma unroll
                for (int j = 0; j < NPT; ++j) {
                    const int64_t gi = g0 + C::jz(j) * plane + (int64_t)C::jy(j) * P.nx + C::jx(j) + lane_off;
                    pv[j] = 0x80;  // outside points act as finished sources
                    tv[j] = inf64();
                    gv[j] = 0.0;
                    mv[j] = 0.0;
                    if (!(lx0 + C::jx(j) < nx && ly0 + C::jy(j) < ny && lz0 + C::jz(j) < nz)) continue;
                    pv[j] = A.par[gi];
                    tv[j] = A.t[gi];
                    gv[j] = A.g[gi];
                    mv[j] = as_f64(__hip_atomic_load((const uint64_t*)A.mu + gi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                }
                int hk = 0;
#pragma unroll
                for (int f = 0; f < C::NF; ++f) {
#pragma unroll
                    for (int b = 0; b < HB[f]; ++b, ++hk) {
                        const int c = lane + b * 64;
                        ht[hk] = inf64();
                        hm[hk] = 0.0;
                        hp[hk] = 0x80;
                        if (((has >> f) & 1) == 0) continue;
                        if (F::cells(f) % 64 != 0 && c >= F::cells(f)) continue;
                        const F e(f, c);
                        if (!(e.lx < nx && e.ly < ny && e.lz < nz)) continue;
                        const int64_t step = f < 2 ? 1 : (f < 4 ? (int64_t)P.nx : plane);
                        const int64_t gi = g0 + e.lz * plane + (int64_t)e.ly * P.nx + e.lx + ((f & 1) ? step : -step);
                        hp[hk] = A.par[gi];
                        ht[hk] = A.t[gi];
                        hm[hk] = as_f64(__hip_atomic_load((const uint64_t*)A.mu + gi, __ATOMIC_RELAXED,
                                                          __HIP_MEMORY_SCOPE_AGENT));
                    }
                }
            }
            for (int i = lane; i < C::NP / 8; i += 64) ((uint64_t*)sF)[i] = 0;
#pragma unroll
            for (int j = 0; j < NPT; ++j) {
                const int L = C::lds(lx0 + C::jx(j), ly0 + C::jy(j), lz0 + C::jz(j));
                const bool src = (pv[j] & 0x80) != 0;
                const bool done = src || !(mv[j] != mv[j]);
                was |= (done ? 1u : 0u) << j;
                sT[L] = tv[j];
                sM[L] = src ? 0.0 : (done ? mv[j] : gv[j]);
                sP[L] = src ? 0x80u | kDone : (pv[j] & 0x3Fu) | (done ? kDone : 0u);
            }
            wave_order();
            // First marks of a later run: a point next to a finished child
            // across a face (nothing inside has changed since the last run).  A
            // first run looks at every point (leaves can sit anywhere).
            int hk = 0;
#pragma unroll
            for (int f = 0; f < C::NF; ++f) {
#pragma unroll
                for (int b = 0; b < HB[f]; ++b, ++hk) {
                    const int c = lane + b * 64;
                    if (F::cells(f) % 64 == 0 || c < F::cells(f)) {
                        const F e(f, c);
                        const int L = e.lds();
                        const bool src = (hp[hk] & 0x80) != 0;
                        const bool done = src || !(hm[hk] != hm[hk]);
                        const uint32_t p = src ? 0x80u | kDone : (hp[hk] & 0x3Fu) | (done ? kDone : 0u);
                        sT[L + F::out(f)] = ht[hk];
                        sM[L + F::out(f)] = src ? 0.0 : hm[hk];
                        sP[L + F::out(f)] = p;
                        // the minus-side neighbour is a child if its plus-side parent is the point
                        const uint32_t want = (f & 1) ? 1u : 2u;
                        if (done && ((p >> (2 * (f >> 1))) & 3u) == want && !(sP[L] & kDone)) sF[e.point()] = 1;
                    }
                }
            }
            wave_order();
        }
        // The octant: per axis, the side most parents of a sample are on.
        int mx, my, mz = 0;
        {
            const uint32_t p = sP[C::lds((lane / C::NCOL) * NPT + NPT / 2, yy, zz)];
            auto minus = [&](int k) {
                return __popcll(__ballot(((p >> (2 * k)) & 3u) == 1u)) > __popcll(__ballot(((p >> (2 * k)) & 3u) == 2u));
            };
            mx = minus(0) ? TX - 1 : 0;
            my = minus(1) ? TY - 1 : 0;
            if (C::D3) mz = minus(2) ? TZ - 1 : 0;
        }
        phase(1);

        // ---- evaluate points whose children are all done, until none is left to look at
        int passes = 0;  // levels with work
        {
            int sweeps = 0;
            bool turn = true, all = !visited;
            uint32_t D = 0;
            int xs = 0, base = 0, pc = 0;
            for (;;) {
                if (turn) {
                    const int cy = yy ^ my, cz = zz ^ mz;
                    base = C::lds(0, cy, cz);
                    pc = (cz * TY + cy) * TX;
                    xs = xs0;
                    D = 0;
                    wave_order();
                    if (all) {
                        D = (1u << NPT) - 1u;
                    } else {
#pragma unroll
                        for (int j = 0; j < NPT; ++j) D |= (uint32_t)sF[pc + (((xs0 + j) & (TX - 1)) ^ mx)] << j;
                    }
                    all = false;
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
                    ++passes;
                    const int L = base + (xs ^ mx);
                    constexpr int NB = C::D3 ? 6 : 4;
                    constexpr int step[6] = {-1, 1, -C::SY, C::SY, -C::SZ, C::SZ};
                    const uint32_t pn = sP[L];
                    uint32_t pm[NB];
#pragma unroll
                    for (int i = 0; i < NB; ++i) pm[i] = sP[L + step[i]];
                    // ready: not done, and no child (a neighbour whose parent on the
                    // side towards the point it is) that is not
                    unsigned long long wait = mask_eq(pn & kDone, kDone);
#pragma unroll
                    for (int i = 0; i < NB; ++i) {
                        const uint32_t want = ((i & 1) ? 1u : 2u) << (2 * (i >> 1)), bits = 3u << (2 * (i >> 1));
                        wait |= mask_eq(pm[i] & (bits | kDone), want);
                    }
                    unsigned long long fin = act & ~wait;
                    unsigned long long a = 0, b = 0;
                    if (fin) {
                        const double tn = sT[L];
                        double lam = sM[L], tm[NB], mm[NB];
#pragma unroll
                        for (int i = 0; i < NB; ++i) {
                            tm[i] = sT[L + step[i]];
                            mm[i] = sM[L + step[i]];
                        }
                        // children in neighbour order x-, x+, y-, y+, z-, z+
#pragma unroll
                        for (int i = 0; i < NB; ++i) {
                            const uint32_t want = ((i & 1) ? 1u : 2u) << (2 * (i >> 1)), bits = 3u << (2 * (i >> 1));
                            const double sum = lam + mm[i] * (tm[i] - tn);
                            lam = in_mask(mask_eq(pm[i] & bits, want)) ? sum : lam;
                        }
                        unsigned long long m1[3] = {0, 0, 0}, m2[3] = {0, 0, 0};  // parent on the minus, plus side
                        double wk[3] = {0.0, 0.0, 0.0};
#pragma unroll
                        for (int i = 0; i < NB / 2; ++i) {
                            m1[i] = mask_eq(pn & (3u << (2 * i)), 1u << (2 * i));
                            m2[i] = mask_eq(pn & (3u << (2 * i)), 2u << (2 * i));
                            const double d = tn - (in_mask(m1[i]) ? tm[2 * i] : tm[2 * i + 1]);
                            wk[i] = in_mask(m1[i] | m2[i]) ? d : 0.0;
                        }
                        double W = wk[0] + wk[1];
                        W = W + wk[2];
                        const double mun = lam / W;
                        fin &= mask_ordered(mun);  // a NaN stays "not done"
                        if (in_mask(fin)) {
                            sM[L] = mun;
                            sP[L] = (uint8_t)(pn | kDone);
                        }
                        // parents inside the tile may now be ready
                        a = (mx ? m1[0] : m2[0]) & fin & __ballot(xs < TX - 1);
                        b = (mx ? m2[0] : m1[0]) & fin & __ballot(xs > 0);
                        a |= ((my ? m1[1] : m2[1]) & fin & aheadY) << 1;
                        b |= ((my ? m2[1] : m1[1]) & fin & behindY) >> 1;
                        if (C::D3) {
                            a |= ((mz ? m1[2] : m2[2]) & fin & (C::NCOL < 64 ? aheadZ : ~0ull)) << TY;
                            b |= ((mz ? m2[2] : m1[2]) & fin & (C::NCOL < 64 ? behindZ : ~0ull)) >> TY;
                        }
                    }
                    // a point behind is next visited by the lane one place back along its column
                    if constexpr (C::NCOL < 64) b = (b >> C::NCOL) | (b << (64 - C::NCOL));
                    D = (D >> 1) | (in_mask(a) ? 1u : 0u) | (in_mask(b) ? 1u << (NPT - 2) : 0u);
                    xs = (xs + 1) & (TX - 1);
                }
                if (quiet) break;
                if (++sweeps > (1 << 20)) {
                    if (lane == 0) set_flag(S, kFlagWatchdog);
                    break;
                }
                // The next sweep turns round along the axes where most lanes' next
                // dirty point has its parent behind.
                int tx2 = 0, ty2 = 0, tz2 = 0;
                {
                    wave_order();
                    const bool any = D != 0u;
                    const uint32_t p = sP[base + (((xs + (any ? __ffs((int)D) - 1 : 0)) & (TX - 1)) ^ mx)];
                    auto turned = [&](int k, int m) {
                        const int n1 = __popcll(__ballot(any && ((p >> (2 * k)) & 3u) == 1u));
                        const int n2 = __popcll(__ballot(any && ((p >> (2 * k)) & 3u) == 2u));
                        return m ? n2 > n1 : n1 > n2;
                    };
                    if (turned(0, mx)) tx2 = TX - 1;
                    if (turned(1, my)) ty2 = TY - 1;
                    if (C::D3 && turned(2, mz)) tz2 = TZ - 1;
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
        if (lane == 0) s_stat[6] += (unsigned long long)passes;
        phase(2);

        // ---- write back newly done points (first run: sources too), gather the faces' keys
        int ndone = 0;
    #pragma unroll
        for (int j = 0; j < NPT; ++j) {
            const int L = C::lds(lx0 + C::jx(j), ly0 + C::jy(j), lz0 + C::jz(j));
            const uint32_t p = sP[L];
            const bool fin = (p & kDone) && !((was >> j) & 1u);
            const bool in = whole || (lx0 + C::jx(j) < nx && ly0 + C::jy(j) < ny && lz0 + C::jz(j) < nz);
            const bool put = fin || (!visited && (p & 0x80u) && in);
            ndone += __popcll(__ballot(fin));
            if (__ballot(put)) {
                const int64_t at = g0 + C::jz(j) * plane + (int64_t)C::jy(j) * P.nx + C::jx(j);
                if (put)
                    __hip_atomic_store((uint64_t*)(A.mu + at) + lane_off, as_u64(sM[L]), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            }
            sF[lane + j * 64] = fin ? 1 : 0;
        }
        wave_order();
        // A face point whose parent lies across that face unblocks the neighbour,
        // keyed by the parent's own time, the earliest bucket in which that
        // parent can be taken (its other children, later in time, are then mostly
        // done as well).
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
                const uint32_t want = (f & 1) ? 2u : 1u;
                const bool on = in && sF[e.point()] != 0 && ((sP[L] >> (2 * (f >> 1))) & 3u) == want;
                const double key = fmax(tref - sT[L + F::out(f)], 0.0);
                fk = on ? nmin(fk, key) : fk;
                any |= __ballot(on);
            }
            if (any) {
                const uint64_t m = wave_min_u64(as_u64(fk));
                if (lane == f) face = m;
            }
        }
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
        stores_done();
        next = uni(publish_wave(S, A.tkey, (uint32_t)tile, slot, !visited, nb, nid, face, true, kInfBits));
        if (lane == 0) s_stat[5] += (unsigned long long)ndone;
        phase(3);
    }
    if (lane == 0) {
        phase(0);
        flush_stats(S, s_stat);
    }
}

}  // namespace eik
