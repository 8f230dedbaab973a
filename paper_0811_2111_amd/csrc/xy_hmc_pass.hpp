// xy_hmc_pass.hpp -- several leap-frog steps of a region in registers.
//
// A workgroup of W waves takes a region of W R rows by 64 entries of a half-row:
// wave w holds rows w R .. w R + R - 1, lane l the two entries of column l (one of
// each colour: the sites 2k and 2k + 1 of the row), angles, momenta and (cos, sin)
// all in registers.  A site's neighbours along the row are the lane's own other
// entry and one entry of the lane beside it (a DPP operand); those above and below
// are the lane's own other-colour entries of the rows beside, which only at a
// wave's first and last row belong to another wave: those two rows of (cos, sin)
// go through LDS, the only LDS traffic of a step, with one barrier (two buffers).
//
// The region is a core grown by K rows above and below and ceil(K / 2) entries on
// either side, taken across the lattice's edges.  Every site of it is updated in
// every step; sites at the rim read lanes and rows outside the region and go wrong
// one site deeper with each step, so after K steps the core is right.  Per site
// the arithmetic is that of k_hmc_step (neighbour sums (left + right) + (up +
// down), the same fma), so the trajectory is bit for bit the one-step one.
//
// Why registers: a pass that keeps (cos, sin) in LDS reads five and writes one
// 8-byte value per site and step, 24 cycles of the CU's LDS for every 64 sites,
// as long as its vector instructions take.  Here a site and step is 15 vector
// instructions instead of 29.
#pragma once

#include "xy_device.hpp"
#include "xy_hmc_site.hpp"
#include "xy_tile1.hpp"

namespace xyd {
namespace hmc {

// Halo of a pass of K steps in entries of a half-row.
__host__ __device__ constexpr int pass_hx(int K) { return (K + 1) / 2; }
// Core of a pass: entries and rows.
__host__ __device__ constexpr int pass_ce(int K) { return 64 - 2 * pass_hx(K); }
template <int W, int R>
__host__ __device__ constexpr int pass_cy(int K) { return W * R - 2 * K; }
template <int W, int R>
__host__ __device__ constexpr int pass_tiles(int L, int K)
{
    return ((L / 2 + pass_ce(K) - 1) / pass_ce(K)) * ((L + pass_cy<W, R>(K) - 1) / pass_cy<W, R>(K));
}
template <int W>
constexpr int kPassLds = 2 * W * 2 * 64;       // float4s: two rows a wave, two buffers

// The value of the lane below (0x138) or above (0x130); lanes at the wave's end read 0.
template <int CTRL>
__device__ __forceinline__ float lane_shift(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
constexpr int kLaneBelow = 0x138, kLaneAbove = 0x130;

template <int R>
struct PassRegs {
    float th[2][R], pm[2][R], c[2][R], s[2][R];
};

// Kick and drift of row r of the wave.  OY: parity of its first row; up, dn: (cos,
// sin) of both colours in the rows above the first and below the last.
template <int R, int OY>
__device__ __forceinline__ void pass_row(PassRegs<R>& g, int r, const float4& up, const float4& dn, float kick,
                                         float drift)
{
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int o = (c + OY + r) & 1, q = 1 - c;
        // left + right: the other colour's entries k - 1, k (o = 0) or k, k + 1
        const float bc = o ? lane_shift<kLaneAbove>(g.c[q][r]) : lane_shift<kLaneBelow>(g.c[q][r]);
        const float bs = o ? lane_shift<kLaneAbove>(g.s[q][r]) : lane_shift<kLaneBelow>(g.s[q][r]);
        const float cu = r > 0 ? g.c[q][r - 1] : (q ? up.z : up.x), su = r > 0 ? g.s[q][r - 1] : (q ? up.w : up.y);
        const float cd = r + 1 < R ? g.c[q][r + 1] : (q ? dn.z : dn.x);
        const float sd = r + 1 < R ? g.s[q][r + 1] : (q ? dn.w : dn.y);
        const float sc = __fadd_rn(__fadd_rn(bc, g.c[q][r]), __fadd_rn(cu, cd));
        const float ss = __fadd_rn(__fadd_rn(bs, g.s[q][r]), __fadd_rn(su, sd));
        const float f = __fmaf_rn(g.s[c][r], sc, -__fmul_rn(g.c[c][r], ss));
        g.pm[c][r] = __fmaf_rn(kick, f, g.pm[c][r]);
        g.th[c][r] = __builtin_amdgcn_fractf(__fmaf_rn(drift, g.pm[c][r], g.th[c][r]));
    }
    __builtin_amdgcn_sched_barrier(0);         // row by row: no sums of later rows kept live
}

template <int R>
__device__ __forceinline__ void pass_cs(PassRegs<R>& g, int r)
{
#pragma unroll
    for (int c = 0; c < 2; ++c) sincos_turn(g.th[c][r], g.s[c][r], g.c[c][r]);
}

// The steps.  A wave publishes its first and last row's (cos, sin) before it updates
// the rows between, which need no other wave, and only then waits for the others:
// the barrier and the LDS latency hide behind those rows.
template <int W, int R, int OY>
__device__ __forceinline__ void pass_steps(PassRegs<R>& g, int K, float kick0, float kick, float drift, int w, int lane,
                                           float4* __restrict__ lds)
{
    static_assert(R % 2 == 0, "every wave's rows start at the same parity");
    const float4 none = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int q = 0; q < K; ++q) {
        float4* buf = lds + (size_t)(q & 1) * (W * 2 * 64);
        const float kq = q == 0 ? kick0 : kick;
        pass_cs<R>(g, 0);
        pass_cs<R>(g, R - 1);
        buf[(2 * w) * 64 + lane] = make_float4(g.c[0][0], g.s[0][0], g.c[1][0], g.s[1][0]);
        buf[(2 * w + 1) * 64 + lane] = make_float4(g.c[0][R - 1], g.s[0][R - 1], g.c[1][R - 1], g.s[1][R - 1]);
#pragma unroll
        for (int r = 1; r < R - 1; ++r) pass_cs<R>(g, r);
#pragma unroll
        for (int r = 1; r < R - 1; ++r) pass_row<R, OY>(g, r, none, none, kq, drift);
        __syncthreads();
        const float4 up = buf[(w > 0 ? 2 * w - 1 : 0) * 64 + lane];
        const float4 dn = buf[(w + 1 < W ? 2 * w + 2 : 2 * w) * 64 + lane];
        pass_row<R, OY>(g, 0, up, none, kq, drift);
        pass_row<R, OY>(g, R - 1, none, dn, kq, drift);
    }
}

__device__ __forceinline__ int pmod(int v, int n)
{
    v %= n;
    return v < 0 ? v + n : v;
}

// K steps of tile b of one lattice, cut into the cores of passes of KH >= K steps;
// kick0: the first step's.  lds: kPassLds<W> entries.
template <int W, int R>
__device__ __forceinline__ void pass_body(const float* __restrict__ src, float* __restrict__ dst,
                                          const float* __restrict__ psrc, float* __restrict__ pdst, int L, int KH,
                                          int K, float kick0, float kick, float drift, int b, float4* lds)
{
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int Hh = L >> 1, hx = pass_hx(KH), CE = pass_ce(KH), CY = pass_cy<W, R>(KH);
    const int tx = (Hh + CE - 1) / CE;
    const int by = b / tx, bx = b - by * tx;
    // the last tiles are moved back inside the lattice
    const int e0 = min(bx * CE, max(Hh - CE, 0)), r0 = min(by * CY, max(L - CY, 0));
    const int k4 = pmod(e0 - hx + lane, Hh) * 4;
    const int yw = r0 - KH + w * R;                // first row, not yet wrapped
    // a descriptor for each plane (below 4 GiB for every L), the row in the scalar offset
    const size_t plane = (size_t)L * (size_t)Hh;
    const unsigned bytes = (unsigned)(plane * 4);
    const __amdgpu_buffer_rsrc_t rs[2] = {make_rsrc(src, bytes), make_rsrc(src + plane, bytes)};
    const __amdgpu_buffer_rsrc_t rp[2] = {make_rsrc(psrc, bytes), make_rsrc(psrc + plane, bytes)};
    PassRegs<R> g;
    unsigned row[R];                               // row offsets in bytes
    int y = pmod(yw, L);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        row[r] = (unsigned)y * (unsigned)(Hh * 4);
        y = y + 1 == L ? 0 : y + 1;
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < 2; ++c)
            g.th[c][r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs[c], k4, (int)row[r], 0));
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < 2; ++c)
            g.pm[c][r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rp[c], k4, (int)row[r], 0));
    // all rows of the workgroup's waves start at the same parity (R and L are even)
    if (yw & 1) pass_steps<W, R, 1>(g, K, kick0, kick, drift, w, lane, lds);
    else pass_steps<W, R, 0>(g, K, kick0, kick, drift, w, lane, lds);
    const __amdgpu_buffer_rsrc_t rd[2] = {make_rsrc(dst, bytes), make_rsrc(dst + plane, bytes)};
    const __amdgpu_buffer_rsrc_t rq[2] = {make_rsrc(pdst, bytes), make_rsrc(pdst + plane, bytes)};
    const int e = lane - hx;                       // core column
    if (e >= 0 && e < CE && e0 + e < Hh) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = w * R + r - KH;          // core row
            if (i >= 0 && i < CY && r0 + i < L) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(g.th[c][r]), rd[c], k4, (int)row[r], 0);
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(g.pm[c][r]), rq[c], k4, (int)row[r], 0);
                }
            }
        }
    }
}

}  // namespace hmc
}  // namespace xyd
