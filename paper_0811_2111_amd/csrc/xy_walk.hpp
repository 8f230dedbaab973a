// xy_walk.hpp -- one sweep of a strip of rows by one wave, everything in registers.
//
// A wave takes 62 pairs of a half-row (its lanes 1 .. 62; lanes 0 and 63 the pairs
// beside them, updated and dropped) and walks down a run of rows.  Step j updates red
// row y0 - 1 + j, then black row y0 - 2 + j, whose red neighbours above, beside and
// below are then new.  The (cos, sin) of the last three rows of either colour stay in
// registers, a neighbour along the row that another lane holds is a DPP operand: no
// LDS, no barrier, no address per neighbour.  The red rows above and below the run
// are updated with their owners' random numbers and not stored, as in a tile; so are
// the red entries in lanes 0 and 63 beside the core.  Rows are loaded D steps ahead;
// row numbers are scalar and enter the buffer instructions as their scalar offset,
// and the lanes and rows that must not be stored get an offset or a descriptor out of
// range, so that no step branches.  Steps are unrolled by six: three rows of (cos,
// sin) and two row parities.
//
// What bounds it: the vector unit, 45 instructions an update, 52 with the halo rows and
// lanes at L = 4096 (256 x 16 tiles: 55), of
// which the eight v_mad_u64_u32 of Philox and the five transcendentals take as long
// as 40 additions; 57 registers, so eight waves a SIMD.  A measured sweep adds every
// black pair's FP32 terms to FP64 sums by itself (88.6 us at L = 6000; 83.0 with FP32
// chains of three rows, which round about three times as much).  Every site goes through
// xyd::site_update with neighbour sums (left + right) + (up + down), so the trajectory
// is that of every other schedule.
#pragma once

#include "xy_tile1.hpp"

namespace xyd {

constexpr int kWalkPairs = 62;

// The value of the lane below (0x138) or above (0x130); the wave's end lanes read 0.
template <int CTRL>
__device__ __forceinline__ float lane_next(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

// Neighbours along the row of the pair (a, b) from the other colour's row `h` =
// (cos, sin) of its entries k, k + 1.  O as in PairNb.
template <int O>
struct WalkSide {
    float2 la, ra, lb, rb;
    __device__ __forceinline__ WalkSide(const float4& h)
    {
        const float2 h0 = make_float2(h.x, h.y), h1 = make_float2(h.z, h.w);
        if constexpr (O) {
            la = h0; ra = h1; lb = h1;
            rb = make_float2(lane_next<0x130>(h.x), lane_next<0x130>(h.y));
        } else {
            la = make_float2(lane_next<0x138>(h.z), lane_next<0x138>(h.w));
            ra = h0; lb = h0; rb = h1;
        }
    }
};

// ST: row loads with the non-temporal hint, for lattices past the last-level cache
// (L = 8192: 117.6 us a sweep against 126.5; on the stores, whose rows share lines
// with the strips beside, it costs: 133).
template <bool MEAS, bool ST>
struct Walk {
    static constexpr int D = 2;       // prefetch depth in rows
    int L, P, y0, n;
    unsigned pitch, half;             // bytes of a half-row, of a half-lattice
    unsigned ldo, sto;                // a lane's byte offset in a half-row: loads, stores
    unsigned pair;
    __amdgpu_buffer_rsrc_t rs, rd, none;
    uint32_t sweep, k0, k1;
    Params p;
    float4 R[3], B[3];                // new red, old black (cos, sin), rows modulo 3
    float2 tr[6], tb[6];              // angles, rows modulo 6
    int acc = 0;
    double v[7] = {0, 0, 0, 0, 0, 0, 0};

    // rows past the run's halo are loaded too, wrapped into the lattice, and never used
    __device__ __forceinline__ unsigned row(int y) const { return (unsigned)wrapi(y, L) * pitch; }
    __device__ __forceinline__ float2 load(unsigned at) const
    {
        return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rs, ldo, at, ST ? kCpolNT : 0));
    }
    __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t r, unsigned at, float a, float b) const
    {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(xu2, make_float2(a, b)), r, sto, at, 0);
    }
    __device__ __forceinline__ float2 load_red(int i) const { return load(row(y0 - 1 + i)); }
    __device__ __forceinline__ float2 load_black(int i) const { return load(half + row(y0 - 2 + i)); }
    static __device__ __forceinline__ float4 cs(float2 t)
    {
        float4 o;
        sincos_turn(t.x, o.y, o.x);
        sincos_turn(t.y, o.w, o.z);
        return o;
    }
    // A black pair's terms into the FP64 sums, gathered as k_measure does, so that a
    // record is k_measure's but for the order of its FP64 sums.
    template <int O>
    __device__ __forceinline__ void measure(const float4& own, const WalkSide<O>& s, const float4& u, const float4& d)
    {
        Meas t{0, 0, 0, 0, 0, 0};
        meas_black(t, own.x, own.y, s.la.x, s.la.y, s.ra.x, s.ra.y, u.x, u.y, d.x, d.y);
        meas_black(t, own.z, own.w, s.lb.x, s.lb.y, s.rb.x, s.rb.y, u.z, u.w, d.z, d.w);
        v[0] += (double)t.cx; v[1] += (double)t.cy; v[2] += (double)t.ix;
        v[3] += (double)t.iy; v[4] += (double)t.mx; v[5] += (double)t.my;
    }
    // One pair: t, own angles and (cos, sin); s, u, d its neighbours; w its random words.
    template <int O>
    __device__ __forceinline__ int update(float2& t, float4& own, const WalkSide<O>& s, const float4& u,
                                          const float4& d, const u32x4& w) const
    {
        const int a = site_update<float>(t.x, own.x, own.y, nsum(s.la.x, s.ra.x, u.x, d.x),
                                         nsum(s.la.y, s.ra.y, u.y, d.y), w.x, w.y, p);
        const int b = site_update<float>(t.y, own.z, own.w, nsum(s.lb.x, s.rb.x, u.z, d.z),
                                         nsum(s.lb.y, s.rb.y, u.w, d.w), w.z, w.w, p);
        return a + b;
    }

    // Red row y0 - 1 + j and, if BLACK (j >= 2), black row y0 - 2 + j.  K = j % 6.
    template <int K, bool BLACK>
    __device__ __forceinline__ void step(int j)
    {
        constexpr int O = (K + 1) & 1;        // y0 is even
        __builtin_amdgcn_sched_barrier(0);    // loads stay ahead of the step before
        tr[(K + D) % 6] = load_red(j + D);
        tb[(K + 2 + D) % 6] = load_black(j + 2 + D);
        const int yr = wrapi(y0 - 1 + j, L), yb = y0 - 2 + j;
        const u32x4 wr = philox10(sweep, 0u, 0u, (uint32_t)yr * (uint32_t)P + pair, k0, k1);
        u32x4 wb;
        if constexpr (BLACK) wb = philox10(sweep, 1u, 0u, (uint32_t)yb * (uint32_t)P + pair, k0, k1);
        B[(K + 2) % 3] = cs(tb[(K + 2) % 6]);
        float2 t = tr[K];
        float4 own = cs(t);
        const int ar = update<O>(t, own, WalkSide<O>(B[(K + 1) % 3]), B[K % 3], B[(K + 2) % 3], wr);
        R[K % 3] = own;
        const bool mine = j <= n && (K != 0 || BLACK);    // not the rows above and below the run
        if (MEAS && mine) acc += ar;
        if (K != 0 || BLACK) store(mine ? rd : none, row(y0 - 1 + j), t.x, t.y);
        if constexpr (BLACK) {
            t = tb[K];
            own = B[K % 3];
            const WalkSide<O> s(R[(K + 2) % 3]);
            const float4 u = R[(K + 1) % 3], d = R[K % 3];
            const int ab = update<O>(t, own, s, u, d, wb);
            store(rd, half + (unsigned)yb * pitch, t.x, t.y);
            if constexpr (MEAS) {
                acc += ab;
                measure<O>(own, s, u, d);
            }
        }
    }

    __device__ __forceinline__ void run()
    {
        static_assert(D == 2);
        tb[0] = load_black(0);
        tb[1] = load_black(1);
        tr[0] = load_red(0);
        tb[2] = load_black(2);
        tr[1] = load_red(1);
        tb[3] = load_black(3);
        B[0] = cs(tb[0]);
        B[1] = cs(tb[1]);
        step<0, false>(0);
        step<1, false>(1);
        for (int j = 2;;) {
            step<2, true>(j);
            if (++j > n + 1) break;
            step<3, true>(j);
            if (++j > n + 1) break;
            step<4, true>(j);
            if (++j > n + 1) break;
            step<5, true>(j);
            if (++j > n + 1) break;
            step<0, true>(j);
            if (++j > n + 1) break;
            step<1, true>(j);
            if (++j > n + 1) break;
        }
        if constexpr (MEAS) v[6] = (double)acc;
    }
};

__host__ __device__ constexpr int walk_strips(int L) { return (L / 4 + kWalkPairs - 1) / kWalkPairs; }

// Strip s of the rows y0 .. y0 + n - 1 (y0 and n even, L % 4 == 0, at least 62 pairs
// a row); the last strip is moved back inside the lattice, where two strips then
// write the same values.  MEAS: the record of the sites of no other strip to part[0 .. 7].
template <bool MEAS, bool ST>
__device__ __forceinline__ void walk_program(const float* __restrict__ src, float* __restrict__ dst, int L, int s,
                                             int y0, int n, uint32_t sweep, uint32_t k0, uint32_t k1, const Params& p,
                                             double* __restrict__ part)
{
    const int lane = threadIdx.x & 63;
    const unsigned bytes = (unsigned)((size_t)L * L * sizeof(float));
    Walk<MEAS, ST> w;
    w.L = L;
    w.P = L >> 2;
    w.y0 = y0;
    w.n = n;
    w.pitch = (unsigned)(L >> 1) * 4u;
    w.half = (unsigned)L * w.pitch;
    const int p0 = min(s * kWalkPairs, w.P - kWalkPairs);
    w.pair = (unsigned)wrapi(p0 - 1 + lane, w.P);
    w.ldo = w.pair * 8u;
    const bool core = lane >= 1 && lane <= kWalkPairs;
    w.sto = core ? w.ldo : 0xfffffff0u;
    w.rs = make_rsrc(src, bytes);
    w.rd = make_rsrc(dst, bytes);
    w.none = make_rsrc(dst, 0u);
    w.sweep = sweep;
    w.k0 = k0;
    w.k1 = k1;
    w.p = p;
    w.run();
    if constexpr (MEAS) {
        const bool mine = core && lane - 1 >= s * kWalkPairs - p0;
#pragma unroll
        for (int q = 0; q < 7; ++q) w.v[q] = mine ? w.v[q] : 0.0;
        wave_record(w.v, part);
    }
}

}  // namespace xyd
