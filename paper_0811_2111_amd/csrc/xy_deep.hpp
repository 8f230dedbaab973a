// xy_deep.hpp -- several sweeps of a small region in one launch, everything on chip.
//
// A workgroup loads a region of the lattice once, keeps its angles and their
// (cos, sin) in registers, a copy of the (cos, sin) of both colours in LDS, runs
// n sweeps on it and writes its core back.  Every thread owns up to R pairs (the
// two entries of one Philox call) of one colour.  A half-sweep reads the other
// colour's (cos, sin) of the neighbours from LDS, updates the own pairs in
// registers and writes their new (cos, sin) to LDS: one barrier per half-sweep
// and no transcendental but those of the proposals.  While one colour's waves
// update, the other's draw the random numbers of their next half-sweep and form
// its proposals, which depend on nothing in LDS; every SIMD holds waves of both colours, so the two
// phases fill each other's latencies.  Lanes are laid out so that a wave's rows
// all have one parity (the position of a site's horizontal neighbours depends
// only on it).
//
// Two forms:
//   WRAP: the region is the whole lattice (at most 4 * 1024 pairs a colour); the
//     LDS planes carry one more row and column on every side, which the owners of
//     the opposite edge keep up to date, so a neighbour's place needs no test.
//     Any number of sweeps.
//   else: the region is a core grown by 2 n sites or more on every side, taken
//     across the lattice's edges.  Sites at the region's rim read places outside
//     it and go wrong, one site deeper with every half-sweep, so that after n
//     sweeps exactly the 2 n outermost sites may be wrong and the core is right.
//     The halo's sites are updated with their owners' random numbers, so no other
//     workgroup's results are needed; src and dst are different buffers.
// ODD: L % 4 == 2, where half-rows have an odd number of entries: the last pair
// of a row has one entry only and pairs beyond the lattice's edge sit at odd
// columns.
//
// What bounds it: the regions of small lattices are one wave a SIMD, and a
// half-sweep is then one chain (LDS read, neighbour sums, exponential, LDS write,
// barrier) of 0.34 us; with several waves a SIMD it is the vector unit (59
// instructions an update at L = 1536, halo included).  Forming the proposals in
// the other colour's half-sweep took L = 128 from 1.47 to 1.36 us a sweep, L = 32 in
// one workgroup from 0.96 to 0.89.
//
// Every site goes through xyd::propose and xyd::decide with neighbour sums
// (left + right) + (up + down), so the trajectory is that of every other schedule.
#pragma once

#include <type_traits>

#include "xy.h"
#include "xy_tile1.hpp"

namespace xyd {

// Region of one workgroup.  Pairs ps .. ps + PC - 1 (modulo P) of the rows ys ..
// ys + RY - 1 (modulo L); its core is cp pairs x cr rows at (hx, hy) inside it.
struct DeepRegion {
    int L, Hh, P;
    int ps, ys;       // in [0, P), [0, L)
    int PC, RY;       // RY even
    int hx, hy, cp, cr;
};

// LDS entries per row of a plane: two columns on either side of the pairs, which
// keeps even columns 16-byte aligned.
__host__ __device__ constexpr int deep_stride(int PC) { return 2 * PC + 4; }
__host__ __device__ constexpr size_t deep_plane(int PC, int RY) { return (size_t)(RY + 2) * deep_stride(PC); }
__host__ __device__ constexpr size_t deep_lds_bytes(int PC, int RY, int nt)
{
    return 2 * deep_plane(PC, RY) * sizeof(float2) + (size_t)(nt / 64) * 7 * sizeof(double);
}

// The two entries of a pair.  The caller's state is aligned to an entry, not
// necessarily to a pair: the copies leave the choice of loads to the compiler.
// Q: entries lie four apart (one replica of a quad's float4 state).
template <typename T, bool Q>
__device__ __forceinline__ float2 pair_ld(const T* e)
{
    if constexpr (Q) return make_float2(store<T>::ld(e[0]), store<T>::ld(e[4]));
    T v[2];
    __builtin_memcpy(v, e, sizeof(v));
    return make_float2(store<T>::ld(v[0]), store<T>::ld(v[1]));
}
template <typename T, bool Q>
__device__ __forceinline__ void pair_st(T* e, float2 f)
{
    if constexpr (Q) {
        e[0] = store<T>::st(f.x);
        e[4] = store<T>::st(f.y);
        return;
    }
    const T v[2] = {store<T>::st(f.x), store<T>::st(f.y)};
    __builtin_memcpy(e, v, sizeof(v));
}

constexpr unsigned kOn = 1, kHasB = 2, kCore = 4, kCol0 = 8, kColN = 16, kRow0 = 32, kRowN = 64;

// Neighbours of the pair whose first entry is plane[at], in the other colour's plane.
template <int O, bool ODD>
__device__ __forceinline__ PairNb<O> deep_nb(const float2* __restrict__ plane, int WS, int at)
{
    PairNb<O> n;
    float2 h0, h1;
    if constexpr (ODD) {
        h0 = plane[at]; h1 = plane[at + 1];
        n.ua = plane[at - WS]; n.ub = plane[at - WS + 1];
        n.da = plane[at + WS]; n.db = plane[at + WS + 1];
    } else {
        const float4 h = *(const float4*)&plane[at];
        const float4 u = *(const float4*)&plane[at - WS];
        const float4 d = *(const float4*)&plane[at + WS];
        h0 = make_float2(h.x, h.y); h1 = make_float2(h.z, h.w);
        n.ua = make_float2(u.x, u.y); n.ub = make_float2(u.z, u.w);
        n.da = make_float2(d.x, d.y); n.db = make_float2(d.z, d.w);
    }
    const float2 side = plane[O ? at + 2 : at - 1];
    n.la = O ? h0 : side;
    n.ra = O ? h1 : h0;
    n.lb = O ? h1 : h0;
    n.rb = O ? side : h1;
    return n;
}

// Pairs whose (cos, sin) a thread keeps in registers beside their angles.  Of eight it
// reads them from LDS, too: 64 registers of state in a workgroup of 1024 threads, which
// has 128, spilled 700 bytes a thread with the neighbours' addresses that the compiler
// kept over the sweeps (L = 128, one sweep 32.0 us, ten 146; without spills 16.1 and 93;
// L = 80, four pairs, ten sweeps 47.0 and 41.2).
constexpr int deep_kept(int R) { return R <= 4 ? R : 1; }

template <int R>
struct DeepItems {
    int at[R];            // first entry within a plane
    unsigned idx[R];      // Philox pair index y * P + p
    unsigned elem[R];     // first entry within a half-lattice
    unsigned flag[R];
};

// How a measured sweep's FP32 terms are gathered before the FP64 sums.  The terms
// and their order are those of the plan that xy_get_plan reports for the lattice,
// so that a record does not depend on the schedule beyond the rounding of FP64
// sums (another order in FP32 shows at 1e-8 of the record at L = 32).
//   kMeasOwn  : a thread's own pairs one after another (the LDS-resident plan);
//   kMeasPair : each pair by itself (k_measure, the streaming plan);
//   kMeasQuad : each pair by itself, in the arithmetic of the tiles (a quad's plan);
//   kMeasChain: columns of `full` pairs, `rp` rows apart, from blocks of rp * full
//               rows (a thread's black pairs in the single-sweep tile), read back
//               from LDS after the black half-sweep.
enum DeepMeas { kMeasNone, kMeasOwn, kMeasPair, kMeasChain, kMeasQuad };

// What a half-sweep can prepare before its neighbours are known, as far as it fits
// into registers beside the angles: with one pair a thread its two proposals; with
// two the random words, with four too where no sums are kept (L = 1000: 4.3 us a
// sweep against 4.7; with sums 6.7 against 6.4); with more nothing.
struct DeepDraw {
    uint32_t sweep, colour, k0, k1;
};
struct DeepProp {
    Proposal a, b;
};
template <int R>
using DeepPrep = std::conditional_t<R == 1, DeepProp, u32x4>;

template <typename T>
__device__ __forceinline__ DeepProp deep_propose(const u32x4& r, float2 th, const Params& p)
{
    return DeepProp{propose<T>(th.x, r.x, r.y, p), propose<T>(th.y, r.z, r.w, p)};
}
template <typename T, int R, bool EARLY>
__device__ __forceinline__ void deep_draw(DeepPrep<R> (&r)[R], const DeepItems<R>& it, const float2 (&th)[R],
                                          const DeepDraw& w, const Params& p)
{
    if constexpr (EARLY)
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const u32x4 v = philox10(w.sweep, w.colour, 0u, it.idx[q], w.k0, w.k1);
            if constexpr (R == 1) r[q] = deep_propose<T>(v, th[q], p);
            else r[q] = v;
        }
}

// The pair's (cos, sin) into its plane; WRAP: and into the rims on the other side.
template <bool ODD, bool WRAP>
__device__ __forceinline__ void deep_put(float2* __restrict__ plane, int WS, int L, int Hh, int at, unsigned flag,
                                         const float4& v)
{
    const bool b = !ODD || (flag & kHasB);
    auto pair = [&](int w) {
        if constexpr (ODD) {
            plane[w] = make_float2(v.x, v.y);
            if (b) plane[w + 1] = make_float2(v.z, v.w);
        } else {
            *(float4*)&plane[w] = v;
        }
    };
    pair(at);
    if constexpr (WRAP) {
        if (flag & (kCol0 | kColN | kRow0 | kRowN)) {
            if (flag & kCol0) plane[at + Hh] = make_float2(v.x, v.y);
            if (flag & kColN) plane[at + (b ? 1 : 0) - Hh] = b ? make_float2(v.z, v.w) : make_float2(v.x, v.y);
            if (flag & kRow0) pair(at + L * WS);
            if (flag & kRowN) pair(at - L * WS);
        }
    }
}

// One half-sweep of this thread's pairs; O = parity (colour + y) & 1 of its rows.
template <typename T, int R, int O, bool ODD, bool WRAP, int MEAS, bool EARLY>
__device__ __forceinline__ void deep_half(float2* __restrict__ own, const float2* __restrict__ oth, int WS, int L,
                                          int Hh, const DeepItems<R>& it, float2 (&th)[R], float4 (&kept)[deep_kept(R)],
                                          DeepPrep<R> (&r)[R], const DeepDraw& w, const Params& p, int& acc, MeasAcc& m, double (&v)[7])
{
#pragma unroll
    for (int q = 0; q < R; ++q) {
        unsigned flag = it.flag[q];
        int at = it.at[q];
        // opaque, so that no addresses derived from them are kept over the sweeps (regions
        // with a halo have the registers, and take 5% longer so)
        if constexpr (WRAP && R >= 4) asm volatile("" : "+v"(flag), "+v"(at));
        if (!(flag & kOn)) continue;
        if constexpr (!EARLY) r[q] = philox10(w.sweep, w.colour, 0u, it.idx[q], w.k0, w.k1);
        const PairNb<O> n = deep_nb<O, ODD>(oth, WS, at);
        float4 copy;                               // (four pairs updated in place spill, too)
        float4& cs = R < 4 ? kept[R < 4 ? q : 0] : copy;
        if constexpr (R == 4) cs = kept[q];
        if constexpr (R > 4) cs = *(const float4*)&own[at];
        DeepProp pr;
        if constexpr (R == 1) pr = r[q];
        else pr = deep_propose<T>(r[q], th[q], p);
        const int aa = decide(pr.a, th[q].x, cs.x, cs.y, nsum(n.la.x, n.ra.x, n.ua.x, n.da.x),
                              nsum(n.la.y, n.ra.y, n.ua.y, n.da.y), p);
        const int ab = decide(pr.b, th[q].y, cs.z, cs.w, nsum(n.lb.x, n.rb.x, n.ub.x, n.db.x),
                              nsum(n.lb.y, n.rb.y, n.ub.y, n.db.y), p);
        deep_put<ODD, WRAP>(own, WS, L, Hh, at, flag, cs);
        if constexpr (R == 4) kept[q] = cs;
        if (flag & kCore) {
            const bool b = !ODD || (flag & kHasB);
            acc += aa + (b ? ab : 0);
            if constexpr (MEAS == kMeasOwn) {
                meas_acc(m, cs.x, cs.y, n.la, n.ra, n.ua, n.da);
                if (b) meas_acc(m, cs.z, cs.w, n.lb, n.rb, n.ub, n.db);
            } else if constexpr (MEAS == kMeasQuad) {
                MeasAcc t;
                meas_acc(t, cs.x, cs.y, n.la, n.ra, n.ua, n.da);
                meas_acc(t, cs.z, cs.w, n.lb, n.rb, n.ub, n.db);
                v[0] += (double)t.cx; v[1] += (double)t.cy; v[2] += (double)t.ix;
                v[3] += (double)t.iy; v[4] += (double)t.mx; v[5] += (double)t.my;
            } else if constexpr (MEAS == kMeasPair) {
                Meas t{0, 0, 0, 0, 0, 0};
                meas_black(t, cs.x, cs.y, n.la.x, n.la.y, n.ra.x, n.ra.y, n.ua.x, n.ua.y, n.da.x, n.da.y);
                if (b)
                    meas_black(t, cs.z, cs.w, n.lb.x, n.lb.y, n.rb.x, n.rb.y, n.ub.x, n.ub.y, n.db.x, n.db.y);
                v[0] += (double)t.cx; v[1] += (double)t.cy; v[2] += (double)t.ix;
                v[3] += (double)t.iy; v[4] += (double)t.mx; v[5] += (double)t.my;
            }
        }
    }
}

// The terms of a measured sweep from the two planes (kMeasChain), this thread's
// share of the core's columns.
template <int NT>
__device__ __forceinline__ void deep_chains(const float2* __restrict__ red, const float2* __restrict__ blk, int WS,
                                            const DeepRegion& g, int rp, int full, double (&v)[7])
{
    for (int c = threadIdx.x; c < g.cp * (g.cr / full); c += NT) {
        const int t = c / g.cp, pc = c - t * g.cp;
        const int bl = t / rp, rt = t - bl * rp;
        MeasAcc m;
        for (int q = 0; q < full; ++q) {
            const int r = g.hy + bl * rp * full + q * rp + rt;
            const int o = (g.ys + r + 1) & 1;
            const int at = (r + 1) * WS + 2 + 2 * (g.hx + pc);
#pragma unroll
            for (int k = at; k < at + 2; ++k)
                meas_acc(m, blk[k].x, blk[k].y, red[k + o - 1], red[k + o], red[k - WS], red[k + WS]);
        }
        v[0] += (double)m.cx; v[1] += (double)m.cy; v[2] += (double)m.ix;
        v[3] += (double)m.iy; v[4] += (double)m.mx; v[5] += (double)m.my;
    }
}

// Pairs of one colour and row parity that NT threads with R pairs each hold: a
// quarter of the threads' share.
template <int NT, int R> constexpr int kDeepPairs = NT / 4 * R;

// n sweeps of region g from src to dst (WRAP: may be the same), the first with
// sweep index sweep0.  me > 0: sweep j (1-based) is measured when (j + phase) % me
// == 0 (rp, full: kMeasChain only); `put(k, s)` is then called by the threads 0 .. 7 for the k-th measured
// sweep of this call (s: their value: six sums, accepts, 0).  smem:
// deep_lds_bytes(PC, RY, NT).
// Q: src and dst are one replica's components of float4 states.
template <typename T, int NT, int R, bool ODD, bool WRAP, int MEAS, bool Q, typename Put>
__device__ __forceinline__ void deep_program(const T* __restrict__ src, T* __restrict__ dst, const DeepRegion& g,
                                             uint32_t sweep0, int n, int me, int phase, int rp, int full, uint32_t k0,
                                             uint32_t k1, const Params& p, char* smem, Put put)
{
    static_assert(NT == 256 || NT % 512 == 0, "waves of both colours and parities");
    static_assert(R <= 4 || !ODD, "own pairs are read from LDS as one");
    constexpr bool EARLY = R <= 2 || (R == 4 && MEAS == kMeasNone);
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // waves are dealt out to the four SIMDs in turn: four red, then four black ones
    const int col = NT == 256 ? w >> 1 : (w >> 2) & 1;
    const int par = w & 1;                        // parity of this wave's region rows
    const int slot = NT == 256 ? 0 : 2 * (w >> 3) + ((w >> 1) & 1);
    const int WS = deep_stride(g.PC);
    float2* red = (float2*)smem;
    float2* blk = red + deep_plane(g.PC, g.RY);
    double* sum = (double*)(blk + deep_plane(g.PC, g.RY));
    float2* own = col ? blk : red;
    const float2* oth = col ? red : blk;
    const unsigned half = col ? (unsigned)(g.L * g.Hh) : 0u;
    DeepItems<R> it;
    float2 th[R];
    float4 kept[deep_kept(R)];
    DeepPrep<R> r[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int i = (q * (NT / 256) + slot) * 64 + lane;      // among the pairs of this colour and parity
        const int ri = i / g.PC, pc = i - ri * g.PC;
        const int rw = 2 * ri + par;
        int y = g.ys + rw, pp = g.ps + pc;
        const bool over = pp >= g.P;
        y = y >= g.L ? y - g.L : y;
        pp = over ? pp - g.P : pp;
        unsigned f = rw < g.RY ? kOn : 0u;
        if (!ODD || pp != g.P - 1) f |= kHasB;
        if (pc >= g.hx && pc < g.hx + g.cp && rw >= g.hy && rw < g.hy + g.cr && rw < g.RY) f |= kCore;
        if constexpr (WRAP) {
            if (pp == 0) f |= kCol0;
            if (pp == g.P - 1) f |= kColN;
            if (y == 0) f |= kRow0;
            if (y == g.L - 1) f |= kRowN;
        }
        it.flag[q] = f;
        it.at[q] = (rw + 1) * WS + 2 + 2 * pc - (ODD && over ? 1 : 0);
        it.idx[q] = (unsigned)(y * g.P + pp);
        it.elem[q] = half + (unsigned)(y * g.Hh + 2 * pp);
        th[q] = make_float2(0.f, 0.f);
        if (f & kOn) {
            const T* e = src + (size_t)it.elem[q] * (Q ? 4 : 1);
            if constexpr (ODD) th[q] = make_float2(store<T>::ld(e[0]), store<T>::ld(e[(f & kHasB) ? 1 : 0]));
            else th[q] = pair_ld<T, Q>(e);
        }
    }
    DeepDraw dr{sweep0, (uint32_t)col, k0, k1};
#pragma unroll
    for (int q = 0; q < R; ++q) {
        float4 made;
        float4& cs = R <= 4 ? kept[R <= 4 ? q : 0] : made;
        sincos_turn(th[q].x, cs.y, cs.x);
        sincos_turn(th[q].y, cs.w, cs.z);
        if (it.flag[q] & kOn) deep_put<ODD, WRAP>(own, WS, g.L, g.Hh, it.at[q], it.flag[q], cs);
    }
    if (col == 0) deep_draw<T, R, EARLY>(r, it, th, dr, p);
    const bool o1 = ((g.ys + par + col) & 1) != 0;     // parity (colour + y) & 1 of this wave's sites (L is even)
    __syncthreads();
    int until = me > 0 ? me - phase % me : 0;     // sweeps up to and with the next measured one
    int rec = 0;
    for (int j = 1; j <= n; ++j) {
        int acc = 0;
        MeasAcc m;
        double v[7] = {0, 0, 0, 0, 0, 0, 0};
        if (col == 0) {
            if (o1) deep_half<T, R, 1, ODD, WRAP, kMeasNone, EARLY>(own, oth, WS, g.L, g.Hh, it, th, kept, r, dr, p, acc, m, v);
            else deep_half<T, R, 0, ODD, WRAP, kMeasNone, EARLY>(own, oth, WS, g.L, g.Hh, it, th, kept, r, dr, p, acc, m, v);
            dr.sweep += 1u;
        } else {
            deep_draw<T, R, EARLY>(r, it, th, dr, p);
        }
        __syncthreads();
        const bool meas = MEAS != kMeasNone && me > 0 && --until == 0;
        if (col == 0) {
            if (j < n) deep_draw<T, R, EARLY>(r, it, th, dr, p);
        } else {
            if (meas) {
                if (o1) deep_half<T, R, 1, ODD, WRAP, MEAS, EARLY>(own, oth, WS, g.L, g.Hh, it, th, kept, r, dr, p, acc, m, v);
                else deep_half<T, R, 0, ODD, WRAP, MEAS, EARLY>(own, oth, WS, g.L, g.Hh, it, th, kept, r, dr, p, acc, m, v);
            } else {
                if (o1) deep_half<T, R, 1, ODD, WRAP, kMeasNone, EARLY>(own, oth, WS, g.L, g.Hh, it, th, kept, r, dr, p, acc, m, v);
                else deep_half<T, R, 0, ODD, WRAP, kMeasNone, EARLY>(own, oth, WS, g.L, g.Hh, it, th, kept, r, dr, p, acc, m, v);
            }
            dr.sweep += 1u;
        }
        if (meas) {
            if constexpr (MEAS == kMeasOwn) {
                v[0] = (double)m.cx; v[1] = (double)m.cy; v[2] = (double)m.ix;
                v[3] = (double)m.iy; v[4] = (double)m.mx; v[5] = (double)m.my;
            }
            if constexpr (MEAS == kMeasChain) {
                __syncthreads();      // the black plane is complete
                deep_chains<NT>(red, blk, WS, g, rp, full, v);
            }
            v[6] = (double)acc;
            const double s = wave_sum7(v);
            const int slot = wave_slot();
            if ((tid & 7) == 0 && slot < 7) sum[w * 7 + slot] = s;
            until = me;
        }
        __syncthreads();
        // the waves' sums, in the order of the waves; they are written again only
        // after the barrier of the next red half-sweep
        if (meas) {
            if (tid < 8) {
                double s = 0.0;
                if (tid < 7)
#pragma unroll
                    for (int k = 0; k < NT / 64; ++k) s += sum[k * 7 + tid];
                put(rec, s);
            }
            ++rec;
        }
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
        if (!(it.flag[q] & kCore)) continue;
        T* e = dst + (size_t)it.elem[q] * (Q ? 4 : 1);
        if constexpr (ODD) {
            e[0] = store<T>::st(th[q].x);
            if (it.flag[q] & kHasB) e[1] = store<T>::st(th[q].y);
        } else {
            pair_st<T, Q>(e, th[q]);
        }
    }
}

}  // namespace xyd
