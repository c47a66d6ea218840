// The block-per-tile kernels: one workgroup per tile, one thread per point, every
// marked point of the tile evaluated once per pass.  They run
//  * the precision ablation's operators, which are not causal;
//  * solves and adjoints of so few tiles that the time of a single run decides
//    (FewTiles, eik_rules.hpp, which has both sides measured).
// The schedule, the tile states and the results are those of the wave-per-tile
// kernels (eik_sweep.hpp, eik_adjoint.hpp).
//
// What bounds them is the chain of passes: a pass is one evaluation of the
// operator (its serial FP64 chain), the LDS reads before it and one barrier,
// about 1.05 us with 1024 threads in 3D and 0.77 us in 2D, however few points are
// marked (a wave's level takes 0.49 and 0.37 us, but a run has three to five times
// as many).  One thread per point, so that no wave has a second evaluation in a
// pass; a tile's waves then fill a compute unit (119 registers, 4 waves per SIMD).
#pragma once

#include "eik_adjoint.hpp"

namespace eik {

// One block's tile in LDS, as far as its kernels share it.
template <int TX, int TY, int TZ>
struct Block {
    using C = SweepCfg<TX, TY, TZ>;
    static constexpr int NT = TX * TY * TZ;
    static constexpr int NF = C::NF;
    static constexpr int NHALO = 2 * (TY * TZ + TX * TZ + (C::D3 ? TX * TY : 0));
    double t[C::NLDS];
    uint8_t dirty[2][NT];
    int more[3];  // per pass (mod 3): some wave marked a point
    int tile, next;
    int64_t slot;
    uint32_t state, nb[6], nid[6];
    unsigned long long face[6];
    unsigned int done;  // points changed by the run
    // statistics: [0..3] phase times on the 100 MHz wall clock (claim, stage,
    // relax, write + publish), [4] visits, [5] point updates, [6] passes, [7]
    // hand-offs, [8] the last phase mark
    unsigned long long stat[9];

    // Thread 0.
    __device__ __forceinline__ void start() {
        next = -1;
        slot = 0;
        for (int i = 0; i < 8; ++i) stat[i] = 0;
        stat[8] = wall_clock64();
    }
    // Thread 0: the time since the last mark goes to phase i.
    __device__ __forceinline__ void phase(int i) {
        const unsigned long long now = wall_clock64();
        stat[i] += now - stat[8];
        stat[8] = now;
    }
    // Claims a tile (or takes the one handed on) and turns it to running; every
    // load of the run comes after.  All threads; the tile is < 0 when none is
    // left, `state` has the skip marker (bit 31) where the visit cap is reached.
    template <int kMaxSleep>
    __device__ __forceinline__ void take(const Sched& S, int32_t& cur_hint) {
        if (threadIdx.x < 64) {
            int64_t sl = slot;
            int ti = next;
            if (ti < 0) ti = claim<kMaxSleep>(S, &sl, cur_hint);
            else if (threadIdx.x == 0) ++stat[7];
            if (threadIdx.x == 0) {
                next = -1;
                tile = ti;
                slot = sl;
                if (ti >= 0) {
                    uint32_t st = __hip_atomic_fetch_xor(S.tstate + ti, kQ | kR, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT);
                    if ((st & (kQ | kR)) != kQ) set_flag(S, kFlagWatchdog);
                    if (S.max_visits > 0) {
                        const unsigned long long v = __hip_atomic_fetch_add(S.counters + 3, 1ull, __ATOMIC_RELAXED,
                                                                            __HIP_MEMORY_SCOPE_AGENT);
                        if ((long long)v >= S.max_visits) {
                            set_flag(S, kFlagLimit);
                            st |= 0x80000000u;
                        }
                    }
                    state = st;
                    done = 0u;
                    more[0] = 0;
                    more[1] = 0;
                    more[2] = 0;
                    ++stat[4];
                    phase(0);
                    stores_done();  // the RMW has returned
                }
            }
        }
        __syncthreads();
    }
    // The face neighbours x-, x+, y-, y+, z-, z+ of the tile (bit 30: it exists).
    __device__ __forceinline__ void neighbours(int ti, int ntx, int nty, int ntz, int tx, int ty, int tz) {
        const int f = threadIdx.x;
        if (f >= 6) return;
        const int d = f >> 1, at = d == 0 ? tx : (d == 1 ? ty : tz), n = d == 0 ? ntx : (d == 1 ? nty : ntz);
        const int step = d == 0 ? 1 : (d == 1 ? ntx : ntx * nty);
        const bool has = (f & 1) ? at < n - 1 : at > 0;
        nb[f] = has ? 0x40000000u : 0u;
        nid[f] = has ? (uint32_t)(ti + ((f & 1) ? step : -step)) : 0u;
        face[f] = kInfBits;
    }
    // Halo cell i: face and cell of it.
    __device__ static __forceinline__ int halo_face(int i, int& c) {
        constexpr int nx = TY * TZ, ny = TX * TZ, nz = TX * TY;
        if (i < 2 * nx) {
            c = i % nx;
            return i / nx;
        }
        i -= 2 * nx;
        if (i < 2 * ny) {
            c = i % ny;
            return 2 + i / ny;
        }
        i -= 2 * ny;
        c = i % nz;
        return 4 + i / nz;
    }
    // The smallest key over the block for face f, of the lanes with `on`.
    __device__ __forceinline__ void face_key(int f, bool on, double key) {
        if (!__ballot(on)) return;
        const uint64_t m = wave_min_u64(as_u64(on ? key : inf64()));
        if ((threadIdx.x & 63) == 0) atomicMin(&face[f], (unsigned long long)m);
    }
    // End of the run: every wave's stores complete before the block hands the
    // tile's faces to the neighbours.
    __device__ __forceinline__ void finish(const Sched& S, uint64_t* tkey, int ti, bool visited, int passes,
                                           unsigned long long self_key) {
        stores_done();
        __syncthreads();
        if (threadIdx.x < 64) {
            const int nxt = publish(S, tkey, (uint32_t)ti, slot, !visited, nb, nid, face, true, self_key);
            if (threadIdx.x == 0) {
                next = nxt;
                stat[5] += done;
                stat[6] += (unsigned long long)passes;
                phase(3);
            }
        }
        __syncthreads();
    }
};

// A forward solve.  OP 0 and 4, the exact operators (uniform and rectilinear):
// values only fall, and a lowered point marks its neighbours above it.  OP 1..3,
// the explicit formulas of the precision ablation (two-dimensional grids): they
// assign their value, which may rise, and are not causal, so every neighbour of a
// changed point is marked (with Sched::track on any change, else on a drop).  The
// marks of a pass go to the other of two flag buffers, so one barrier per pass
// orders them before the next pass's reads.
template <int TX, int TY, int TZ, int OP>
__global__ void __launch_bounds__(TX* TY* TZ) k_block(SolveArgs A) {
    using B = Block<TX, TY, TZ>;
    using C = SweepCfg<TX, TY, TZ>;
    using F = Face<TX, TY, TZ>;
    constexpr int NT = B::NT;
    constexpr bool kExact = OP == 0 || OP == 4;
    static_assert(kExact || TZ == 1, "the ablation operators are two-dimensional");
    __shared__ B s;
    __shared__ unsigned long long s_pend;                   // smallest value held back by the horizon
    __shared__ double sW[OP == 4 ? 2 * (TX + TY + TZ) : 1];  // reciprocal spacings, as in k_sweep

    const int tid = threadIdx.x, lane = tid & 63;
    const int lx = tid % TX, ly = (tid / TX) % TY, lz = tid / (TX * TY), L = C::lds(lx, ly, lz);
    double* const sT = s.t;
    const Sched& S = A.s;
    if (tid == 0) s.start();
    int32_t cur_hint = 0;  // wave 0: the window's lowest bucket as last seen
    for (;;) {
        s.template take<kExact ? 1 : 8>(S, cur_hint);
        const int tile = s.tile;
        if (tile < 0) break;
        const uint32_t st = s.state;
        if (st & 0x80000000u) {  // visit cap reached: drop the tile
            if (tid == 0) drop_run(S, (uint32_t)tile, s.slot);
            __syncthreads();
            continue;
        }
        const bool visited = (st & kV) != 0;
        const Prob P = wave_prob_of_tile(A.pt, uni(tile));
        const int tl = tile - P.tile_off;
        const int tx = tl % P.ntx, ty = (tl / P.ntx) % P.nty, tz = tl / (P.ntx * P.nty);
        const int x0 = tx * TX, y0 = ty * TY, z0 = tz * TZ;
        const double hz = (double)(slot_bucket(s.slot) + S.horizon);  // horizon, as in k_sweep
        s.neighbours(tile, P.ntx, P.nty, P.ntz, tx, ty, tz);
        if (tid == 0) s_pend = kInfBits;
        // ---- stage the tile and its halo -----------------------------------
        const int x = x0 + lx, y = y0 + ly, z = z0 + lz;
        const bool in = x < P.nx && y < P.ny && z < P.nz;
        const int64_t plane = (int64_t)P.ny * P.nx;
        const int64_t gi = P.pt_off + z * plane + (int64_t)y * P.nx + x;
        double q = 0.0, t_in = inf64();
        bool src = false;
        if (in) {
            bool ok;
            q = field_q(A.field[gi], P.h, P.kind, ok);
            t_in = as_f64(__hip_atomic_load((const uint64_t*)(A.t + gi), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            if (!ok) set_flag(S, kFlagDomain);
            src = signbit(t_in);
            if (!ok || src) q = 0.0;  // a source is fixed
            t_in = fabs(t_in);
        }
        sT[L] = t_in;
        for (int i = tid; i < B::NHALO; i += NT) {
            int c;
            const int f = B::halo_face(i, c), side = (f & 1) ? 1 : -1;
            const F e(f, c);
            const int X = x0 + e.lx + (f < 2 ? side : 0), Y = y0 + e.ly + (f >> 1 == 1 ? side : 0);
            const int Z = z0 + e.lz + (f >= 4 ? side : 0);
            const bool hin = X >= 0 && X < P.nx && Y >= 0 && Y < P.ny && Z >= 0 && Z < P.nz;
            sT[e.lds() + F::out(f)] = hin ? hload(A.t + P.pt_off + Z * plane + (int64_t)Y * P.nx + X) : inf64();
        }
        if constexpr (OP == 4) {
            constexpr int NW = 2 * (TX + TY + TZ);
            for (int i = tid; i < NW; i += NT) {
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
        s.dirty[0][tid] = 0;
        s.dirty[1][tid] = 0;
        __syncthreads();
        // first pass: every point on a first run, in a tile holding a source and
        // with a horizon; otherwise boundary points next to a halo value below
        // their own
        bool dirty = !visited || (st & kS) || S.horizon > 0;
        if (!dirty) {
            dirty = (lx == 0 && sT[L - 1] < t_in) || (lx == TX - 1 && sT[L + 1] < t_in) ||
                    (ly == 0 && sT[L - C::SY] < t_in) || (ly == TY - 1 && sT[L + C::SY] < t_in);
            if (C::D3) dirty = dirty || (lz == 0 && sT[L - C::SZ] < t_in) || (lz == TZ - 1 && sT[L + C::SZ] < t_in);
        }
        if (tid == 0) s.phase(1);
        // ---- relax until the tile is quiet ---------------------------------
        int cb = 0, passes = 0;
        double v = t_in, pend = inf64();
        for (;;) {
            if (tid == 0) s.more[(passes + 1) % 3] = 0;  // written next pass; last read two barriers ago
            bool marked = false;
            const unsigned long long act = __ballot(dirty && q > 0.0);
            if (act) {
                const double xa = sT[L - 1], xb = sT[L + 1], ya = sT[L - C::SY], yb = sT[L + C::SY];
                const double za = C::D3 ? sT[L - C::SZ] : inf64(), zb = C::D3 ? sT[L + C::SZ] : inf64();
                double r;
                bool ch;
                if constexpr (OP == 0) {
                    r = update_short<C::D3>(nmin(xa, xb), nmin(ya, yb), nmin(za, zb), q, v, act);
                    ch = r < v;
                } else if constexpr (OP == 4) {
                    const double n6[6] = {xa, xb, ya, yb, za, zb};
                    const double w6[6] = {sW[lx], sW[TX + lx], sW[2 * TX + ly], sW[2 * TX + TY + ly],
                                          C::D3 ? sW[2 * (TX + TY) + lz] : 1.0, C::D3 ? sW[2 * (TX + TY) + TZ + lz] : 1.0};
                    r = update_rect_short<C::D3>(n6, w6, q, v, act);
                    ch = r < v;
                } else {
                    r = apply_op<OP>(nmin(xa, xb), nmin(ya, yb), inf64(), q);
                    ch = r != v && r == r;
                }
                ch = ch && in_mask(act);
                if (kExact && S.horizon > 0) {
                    const double rb = r * S.inv_delta;
                    if (ch && rb >= hz && rb < 1.0e15) {
                        pend = nmin(pend, r);
                        ch = false;
                    }
                }
                marked = ch && (kExact || S.track || r < v);
                if (ch) {
                    v = r;
                    sT[L] = r;
                }
                if (marked) {
                    uint8_t* nd = s.dirty[cb ^ 1];
                    if (lx > 0 && (!kExact || xa > r)) nd[tid - 1] = 1;
                    if (lx < TX - 1 && (!kExact || xb > r)) nd[tid + 1] = 1;
                    if (ly > 0 && (!kExact || ya > r)) nd[tid - TX] = 1;
                    if (ly < TY - 1 && (!kExact || yb > r)) nd[tid + TX] = 1;
                    if (C::D3) {
                        if (lz > 0 && za > r) nd[tid - TX * TY] = 1;
                        if (lz < TZ - 1 && zb > r) nd[tid + TX * TY] = 1;
                    }
                }
            }
            if (__ballot(marked) && lane == 0) s.more[passes % 3] = 1;
            __syncthreads();
            const int more = s.more[passes % 3];
            ++passes;
            if (!more) break;
            cb ^= 1;
            dirty = s.dirty[cb][tid] != 0;
            s.dirty[cb][tid] = 0;
            if (passes >= (kExact ? 1 << 20 : 1 << 16)) {  // the ablation operators need not settle
                if (tid == 0) set_flag(S, kExact ? kFlagWatchdog : kFlagLimit);
                break;
            }
        }
        if (tid == 0) s.phase(2);
        // ---- write back changed points, gather the faces' minima -----------
        // A source counts on the first run (it is never lowered).  With an exact
        // operator a face value matters where it is below the neighbour's own value
        // across the face, otherwise (not causal) every lowered one does, and a
        // raised one with tracking.
        const bool chg = in && v != t_in;
        const bool live = (chg && (v < t_in || S.track)) || (src && !visited);
        if (chg) tstore(A.t + gi, v);
        const bool on[6] = {lx == 0, lx == TX - 1, ly == 0, ly == TY - 1, lz == 0, lz == TZ - 1};
#pragma unroll
        for (int f = 0; f < B::NF; ++f)
            s.face_key(f, live && on[f] && (!kExact || v < sT[on[f] ? L + F::out(f) : L]), v);
        const int cnt = __popcll(__ballot(chg));
        if (cnt && lane == 0) atomicAdd(&s.done, (unsigned int)cnt);
        unsigned long long self_key = kInfBits;
        if (kExact && S.horizon > 0) {
            if (__ballot(pend < inf64())) {
                const double m = wave_min(pend);
                if (lane == 0) atomicMin(&s_pend, (unsigned long long)as_u64(m));
            }
            __syncthreads();
            self_key = s_pend;
        }
        s.finish(S, A.tkey, tile, visited, passes, self_key);
    }
    if (tid == 0) {
        s.phase(0);
        flush_stats(S, s.stat);
    }
}

// An adjoint: a point is evaluated when all its children are done, and marks its
// parents in the tile for the next pass (rules and results as in k_adjoint).
template <int TX, int TY, int TZ>
__global__ void __launch_bounds__(TX* TY* TZ) k_adjoint_block(AdjArgs A) {
    using B = Block<TX, TY, TZ>;
    using C = SweepCfg<TX, TY, TZ>;
    using F = Face<TX, TY, TZ>;
    constexpr int NT = B::NT, NB = C::NF;
    __shared__ B s;
    __shared__ double sM[C::NLDS];   // mu, NaN where it is not done
    __shared__ uint8_t sP[C::NLDS];  // parent codes, 0x80 a source or outside the grid

    const int tid = threadIdx.x, lane = tid & 63;
    const int lx = tid % TX, ly = (tid / TX) % TY, lz = tid / (TX * TY), L = C::lds(lx, ly, lz);
    const Sched& S = A.s;
    const double tref = as_f64(*A.tref_bits);
    if (tid == 0) s.start();
    int32_t cur_hint = 0;
    for (;;) {
        s.template take<1>(S, cur_hint);
        const int tile = s.tile;
        if (tile < 0) break;
        const bool visited = (s.state & kV) != 0;
        const Prob P = wave_prob_of_tile(A.pt, uni(tile));
        const int tl = tile - P.tile_off;
        const int tx = tl % P.ntx, ty = (tl / P.ntx) % P.nty, tz = tl / (P.ntx * P.nty);
        const int x0 = tx * TX, y0 = ty * TY, z0 = tz * TZ;
        s.neighbours(tile, P.ntx, P.nty, P.ntz, tx, ty, tz);
        // ---- stage the tile and its halo: outside cells act as finished sources
        const int64_t plane = (int64_t)P.ny * P.nx;
        const int x = x0 + lx, y = y0 + ly, z = z0 + lz;
        const bool in = x < P.nx && y < P.ny && z < P.nz;
        const int64_t gi = P.pt_off + z * plane + (int64_t)y * P.nx + x;
        uint32_t pn = 0x80u;
        double tn = inf64(), gn = 0.0, mu = 0.0;
        if (in) {
            pn = A.par[gi];
            tn = A.t[gi];
            gn = A.g[gi];
            mu = as_f64(__hip_atomic_load((const uint64_t*)(A.mu + gi), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            if (pn & 0x80u) mu = 0.0;
        }
        s.t[L] = tn;
        sM[L] = mu;
        sP[L] = (uint8_t)pn;
        for (int i = tid; i < B::NHALO; i += NT) {
            int c;
            const int f = B::halo_face(i, c), side = (f & 1) ? 1 : -1;
            const F e(f, c);
            const int X = x0 + e.lx + (f < 2 ? side : 0), Y = y0 + e.ly + (f >> 1 == 1 ? side : 0);
            const int Z = z0 + e.lz + (f >= 4 ? side : 0);
            double ht = inf64(), hm = 0.0;
            uint32_t hp = 0x80u;
            if (X >= 0 && X < P.nx && Y >= 0 && Y < P.ny && Z >= 0 && Z < P.nz) {
                const int64_t hi = P.pt_off + Z * plane + (int64_t)Y * P.nx + X;
                hp = A.par[hi];
                ht = A.t[hi];
                hm = as_f64(__hip_atomic_load((const uint64_t*)(A.mu + hi), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                if (hp & 0x80u) hm = 0.0;
            }
            const int H = e.lds() + F::out(f);
            s.t[H] = ht;
            sM[H] = hm;
            sP[H] = (uint8_t)hp;
        }
        s.dirty[0][tid] = 0;
        s.dirty[1][tid] = 0;
        __syncthreads();
        const bool was = !(mu != mu);
        bool done = was;
        // first run: every point (leaves can sit anywhere); later runs: the
        // boundary, since readiness can only come from children across a face
        bool dirty = !visited || lx == 0 || lx == TX - 1 || ly == 0 || ly == TY - 1 ||
                     (C::D3 && (lz == 0 || lz == TZ - 1));
        if (tid == 0) s.phase(1);
        int cb = 0, passes = 0;
        constexpr int step[6] = {-1, 1, -C::SY, C::SY, -C::SZ, C::SZ};
        constexpr int pstep[6] = {-1, 1, -TX, TX, -TX * TY, TX * TY};
        for (;;) {
            if (tid == 0) s.more[(passes + 1) % 3] = 0;
            bool marked = false;
            if (dirty && !done) {
                uint32_t pm[NB];
                double mm[NB], tm[NB];
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    pm[i] = sP[L + step[i]];
                    mm[i] = sM[L + step[i]];
                    tm[i] = s.t[L + step[i]];
                }
                bool ready = true;
                double lam = gn;
                // children in neighbour order x-, x+, y-, y+, z-, z+: a neighbour whose
                // parent lies on the side towards this point
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    if (!(pm[i] & 0x80u) && ((pm[i] >> (2 * (i >> 1))) & 3u) == ((i & 1) ? 1u : 2u)) {
                        if (mm[i] != mm[i]) ready = false;
                        const double w = tm[i] - tn;
                        lam = lam + mm[i] * w;
                    }
                }
                if (ready) {
                    double wk[3] = {0.0, 0.0, 0.0};
#pragma unroll
                    for (int i = 0; i < NB / 2; ++i) {
                        const uint32_t code = (pn >> (2 * i)) & 3u;
                        if (code == 1u) wk[i] = tn - tm[2 * i];
                        else if (code == 2u) wk[i] = tn - tm[2 * i + 1];
                    }
                    double W = wk[0] + wk[1];
                    W = W + wk[2];
                    const double mun = lam / W;
                    if (mun == mun) {  // a NaN stays "not done"
                        mu = mun;
                        sM[L] = mun;
                        done = true;
                        uint8_t* nd = s.dirty[cb ^ 1];
                        const bool room[6] = {lx > 0, lx < TX - 1, ly > 0, ly < TY - 1, lz > 0, lz < TZ - 1};
#pragma unroll
                        for (int i = 0; i < NB; ++i) {
                            if (((pn >> (2 * (i >> 1))) & 3u) == ((i & 1) ? 2u : 1u) && room[i]) {
                                nd[tid + pstep[i]] = 1;
                                marked = true;
                            }
                        }
                    }
                }
            }
            if (__ballot(marked) && lane == 0) s.more[passes % 3] = 1;
            __syncthreads();
            const int more = s.more[passes % 3];
            ++passes;
            if (!more) break;
            cb ^= 1;
            dirty = s.dirty[cb][tid] != 0;
            s.dirty[cb][tid] = 0;
            if (passes >= (1 << 20)) {
                if (tid == 0) set_flag(S, kFlagWatchdog);
                break;
            }
        }
        if (tid == 0) s.phase(2);
        // ---- write back newly done points (first run: sources too) and the faces'
        // keys: the time of the parent across the face
        const bool fin = done && !was;
        if (fin || (!visited && in && (pn & 0x80u)))
            __hip_atomic_store((uint64_t*)(A.mu + gi), as_u64(mu), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const bool on[6] = {lx == 0, lx == TX - 1, ly == 0, ly == TY - 1, lz == 0, lz == TZ - 1};
#pragma unroll
        for (int f = 0; f < B::NF; ++f) {
            const bool up = fin && on[f] && ((pn >> (2 * (f >> 1))) & 3u) == ((f & 1) ? 2u : 1u);
            s.face_key(f, up, up ? fmax(tref - s.t[L + F::out(f)], 0.0) : 0.0);
        }
        const int cnt = __popcll(__ballot(fin));
        if (cnt && lane == 0) atomicAdd(&s.done, (unsigned int)cnt);
        s.finish(S, A.tkey, tile, visited, passes, kInfBits);
    }
    if (tid == 0) {
        s.phase(0);
        flush_stats(S, s.stat);
    }
}

}  // namespace eik
