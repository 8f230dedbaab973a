// xy_hmc.hip -- hybrid Monte Carlo trajectories (section 1.2): Gaussian momenta,
// leap-frog integration of the equations of motion, Metropolis step on FP64
// global sums of H = sum p^2/2 + beta E, all on the device.
//
// Angles are in turns (phi = theta / 2 pi), momenta in radians per unit time,
// both FP32 in the half-lattice layout of the state.  With
//     F_i = -beta sum_{j nn i} sin(theta_i - theta_j)
//         = -beta (s_i sum_j c_j - c_i sum_j s_j),   (c, s) = (cos, sin) theta,
// one trajectory of n leap-frog steps of size eps is
//     begin : p = Box-Muller(Philox), saved = phi, H_old partials;
//     step 1: p += eps/2 F(phi), phi += eps/(2 pi) p     (kick, then drift)
//     step k: p += eps   F(phi), phi += eps/(2 pi) p     (k = 2 .. n; two half
//             kicks of neighbouring steps merged)
//     end   : p += eps/2 F(phi), H_new partials;
//     decide: dH = H_new - H_old (FP64), accept iff u < exp(-dH);
//     restore phi = saved if rejected.
// A step is a Jacobi update (every site from the same old angles), so the
// angles ping-pong between the state and a second buffer; momenta are local and
// are updated in place.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "xy_device.hpp"
#include "xy_hmc_pass.hpp"
#include "xy_hmc_site.hpp"
#include "xy_launch.hpp"
#include "xy_reduce.hpp"

using namespace xyd;
using namespace xyd::hmc;

namespace xyk {

namespace {

constexpr int kThreads = 256;

// The angle of entry (c, y, k) and the (cos, sin) of it and of its four
// neighbours in the other plane.
__device__ __forceinline__ Nb load_nb(const float* __restrict__ st, int L, int Hh, int c, int y, int k, float& th)
{
    const int o = (c + y) & 1;
    const float* oth = st + (size_t)(1 - c) * L * Hh;
    th = st[((size_t)c * L + y) * Hh + k];
    const float tl = oth[(size_t)y * Hh + wrapi(k + o - 1, Hh)];
    const float tr = oth[(size_t)y * Hh + wrapi(k + o, Hh)];
    const float tu = oth[(size_t)wrapi(y - 1, L) * Hh + k];
    const float td = oth[(size_t)wrapi(y + 1, L) * Hh + k];
    Nb n;
    sincos_turn(th, n.s, n.c);
    sincos_turn(tl, n.sl, n.cl);
    sincos_turn(tr, n.sr, n.cr);
    sincos_turn(tu, n.su, n.cu);
    sincos_turn(td, n.sd, n.cd);
    return n;
}

// One partial record per wave: (Cx, Cy, Ix, Iy, Mx, My, K, 0).  Black sites add
// their four bonds, their own spin and that of the red site to their right (as
// the Metropolis measurement does); every site adds p^2 / 2.
__device__ __forceinline__ void write_record(const double (&v)[7], double* __restrict__ rec, unsigned b)
{
    wave_record(v, rec + ((size_t)b * (kThreads / 64) + (threadIdx.x >> 6)) * 8);
}

__device__ __forceinline__ void accumulate(double v[7], const Nb& n, int c, float kin)
{
    if (c == 1) {
        Meas m{0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        meas_black(m, n.c, n.s, n.cl, n.sl, n.cr, n.sr, n.cu, n.su, n.cd, n.sd);
        v[0] += (double)m.cx; v[1] += (double)m.cy; v[2] += (double)m.ix;
        v[3] += (double)m.iy; v[4] += (double)m.mx; v[5] += (double)m.my;
    }
    v[6] += (double)kin;
}

// Workgroups are dispatched round-robin over the 8 XCDs (block b -> XCD b % 8);
// this remap gives each XCD one contiguous band of rows (both colours), so the
// neighbour rows a block reads from the other plane are hits in that XCD's L2.
__device__ __forceinline__ unsigned xcd_band(unsigned b, unsigned nb)
{
    if ((nb & 7u) != 0u) return b;
    return (b & 7u) * (nb >> 3) + (b >> 3);
}

// Whether the trajectory before this one in the same call was rejected: its begin
// kernel's saved angles then are the state, which holds the rejected ones.  The
// begin reads them there and writes them to the state, in place of the other way
// round: a launch of 4.8 us a trajectory less than a copy back after each.
__device__ __forceinline__ bool rejected_before(int again, const unsigned* flag) { return again && flag[0] == 0u; }

// Record-writing passes: 1-D grid of cols x rb workgroups, cols = 2 ceil(Hh/256)
// (column block, colour interleaved), rb row blocks; after the XCD remap t,
// column t % cols takes the run of R = ceil(L / rb) consecutive rows starting at
// (t / cols) R, so the rows above and the row itself that a thread needs from
// the other plane were loaded in its previous iteration.  Record index: t.
//
// Momenta, saved angles and the partial records of H_old.
__global__ void __launch_bounds__(kThreads)
k_hmc_begin(float* st, float* __restrict__ p, float* copy, int L, uint32_t traj,
            uint32_t k0, uint32_t k1, int cols, int rb, int again, unsigned* __restrict__ flag, double* __restrict__ rec)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) flag[1] = 0u;
    const bool back = rejected_before(again, flag);
    const float* from = back ? copy : st;
    float* saved = back ? st : copy;
    const int Hh = L >> 1, P = (Hh + 1) >> 1;
    const unsigned t = xcd_band(blockIdx.x, gridDim.x);
    const int col = (int)(t % (unsigned)cols);
    const int k = (col >> 1) * kThreads + threadIdx.x;
    const int c = col & 1;
    double v[7] = {0, 0, 0, 0, 0, 0, 0};
    const int R = (L + rb - 1) / rb, y0 = (int)(t / (unsigned)cols) * R, y1 = y0 + R < L ? y0 + R : L;
    if (k < Hh) {
        for (int y = y0; y < y1; ++y) {
            float th;
            const Nb n = load_nb(from, L, Hh, c, y, k, th);
            const size_t i = ((size_t)c * L + y) * Hh + k;
            saved[i] = th;
            const u32x4 r = philox10(traj, (uint32_t)c, 2u, (uint32_t)y * (uint32_t)P + (uint32_t)(k >> 1), k0, k1);
            const float pm = (k & 1) ? box_muller(r.z, r.w) : box_muller(r.x, r.y);
            p[i] = pm;
            accumulate(v, n, c, __fmul_rn(0.5f, __fmul_rn(pm, pm)));
        }
    }
    write_record(v, rec, t);              // every lane reaches the wave sums
}

// One leap-frog step: kick with `kick` = eps (eps/2 on the first step), then
// drift by eps/(2 pi) p turns.  Grid (2 ceil(Hh/256), L).
__global__ void __launch_bounds__(kThreads)
k_hmc_step(const float* __restrict__ src, float* __restrict__ dst, float* __restrict__ p, int L, float nbeta_kick,
           float drift)
{
    const int Hh = L >> 1;
    const int k = (blockIdx.x >> 1) * kThreads + threadIdx.x;
    if (k >= Hh) return;
    const int y = blockIdx.y, c = blockIdx.x & 1;
    float th;
    const Nb n = load_nb(src, L, Hh, c, y, k, th);
    const size_t i = ((size_t)c * L + y) * Hh + k;
    const float pn = __fmaf_rn(nbeta_kick, sin_sum(n), p[i]);
    p[i] = pn;
    dst[i] = __builtin_amdgcn_fractf(__fmaf_rn(drift, pn, th));
}

// One leap-frog step for L % 4 == 0: a thread takes the two entries 2j, 2j+1 of
// a half-row in R consecutive rows (8-byte loads and stores).  Its horizontal
// neighbours in the other plane are that plane's pair 2j, 2j+1 of the same row
// and one more entry (2j-1 if o = 0, 2j+2 if o = 1); its vertical neighbours are
// the other plane's pairs of the rows above and below, so the R rows share R + 2
// rows of the other plane.  step2_blocks(L) workgroups, t after the XCD remap.
constexpr int kStepRows = 4;
__host__ __device__ constexpr unsigned step2_blocks(int L)
{
    return 2u * (((unsigned)(L / 4) + kThreads - 1) / kThreads) * (unsigned)(L / kStepRows);
}
template <int R>
__device__ __forceinline__ void step2_body(const float* __restrict__ src, float* __restrict__ dst,
                                           float* __restrict__ p, int L, float nbeta_kick, float drift, unsigned t)
{
    const int Hh = L >> 1, J = Hh >> 1;
    const int cols = 2 * ((J + kThreads - 1) / kThreads);
    const int y0 = (int)(t / (unsigned)cols) * R, col = (int)(t % (unsigned)cols);
    const int c = col & 1;
    const int j = (col >> 1) * kThreads + threadIdx.x;
    if (j >= J) return;
    const float* oth = src + (size_t)(1 - c) * L * Hh;
    float2 h[R + 2];                       // other plane, rows y0-1 .. y0+R
#pragma unroll
    for (int r = 0; r < R + 2; ++r) h[r] = ((const float2*)(oth + (size_t)wrapi(y0 - 1 + r, L) * Hh))[j];
    float2 th[R], pv[R];
    float e[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int y = y0 + r;
        const int o = (c + y) & 1;
        th[r] = ((const float2*)(src + ((size_t)c * L + y) * Hh))[j];
        pv[r] = ((const float2*)(p + ((size_t)c * L + y) * Hh))[j];
        e[r] = oth[(size_t)y * Hh + (o ? wrapi(2 * j + 2, Hh) : wrapi(2 * j - 1, Hh))];
    }
    float hc0[R + 2], hs0[R + 2], hc1[R + 2], hs1[R + 2];
#pragma unroll
    for (int r = 0; r < R + 2; ++r) {
        sincos_turn(h[r].x, hs0[r], hc0[r]);
        sincos_turn(h[r].y, hs1[r], hc1[r]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int y = y0 + r;
        const int o = (c + y) & 1;
        float sa, ca, sb, cb, se, ce;
        sincos_turn(th[r].x, sa, ca);
        sincos_turn(th[r].y, sb, cb);
        sincos_turn(e[r], se, ce);
        Nb na, nb;
        na.c = ca; na.s = sa;
        nb.c = cb; nb.s = sb;
        // entry 2j: left = (o ? h0 : e), right = (o ? h1 : h0); 2j+1: left = (o ? h1 : h0), right = (o ? e : h1)
        na.cl = o ? hc0[r + 1] : ce;         na.sl = o ? hs0[r + 1] : se;
        na.cr = o ? hc1[r + 1] : hc0[r + 1]; na.sr = o ? hs1[r + 1] : hs0[r + 1];
        nb.cl = o ? hc1[r + 1] : hc0[r + 1]; nb.sl = o ? hs1[r + 1] : hs0[r + 1];
        nb.cr = o ? ce : hc1[r + 1];         nb.sr = o ? se : hs1[r + 1];
        na.cu = hc0[r]; na.su = hs0[r]; nb.cu = hc1[r]; nb.su = hs1[r];
        na.cd = hc0[r + 2]; na.sd = hs0[r + 2]; nb.cd = hc1[r + 2]; nb.sd = hs1[r + 2];
        const float pa = __fmaf_rn(nbeta_kick, sin_sum(na), pv[r].x);
        const float pb = __fmaf_rn(nbeta_kick, sin_sum(nb), pv[r].y);
        ((float2*)(p + ((size_t)c * L + y) * Hh))[j] = make_float2(pa, pb);
        ((float2*)(dst + ((size_t)c * L + y) * Hh))[j] =
            make_float2(__builtin_amdgcn_fractf(__fmaf_rn(drift, pa, th[r].x)),
                        __builtin_amdgcn_fractf(__fmaf_rn(drift, pb, th[r].y)));
    }
}

__global__ void __launch_bounds__(kThreads)
k_hmc_step2(const float* __restrict__ src, float* __restrict__ dst, float* __restrict__ p, int L, float nbeta_kick,
            float drift)
{
    step2_body<kStepRows>(src, dst, p, L, nbeta_kick, drift, xcd_band(blockIdx.x, gridDim.x));
}

// Several leap-frog steps per pass (xy_hmc_pass.hpp) for any even L: 512 threads,
// eight rows a thread (64 x 128 sites a region; 104 VGPRs, two workgroups a CU), or
// four while those regions are about one a CU, when a pass is as long as one wave's
// work (L = 512, 145 regions: 7.6 us against 11.5; L = 1024, 570 regions: 13.9
// against 11.5).
// A pass of 7 steps, eight rows: L = 4096 90 us, L = 8192 325 us (64 x 64 tiles with
// (cos, sin) in LDS: 134 and 503); four rows: L = 256 6.4 us (12.4).  Other shapes at
// L = 4096, 7 steps: 12 waves of six rows 95 us, 16 of four 97, 16 of eight 117 (one
// workgroup a CU).
constexpr int kMaxStepsPerPass = 8;
// Steps of a trajectory's longest pass: the fewest passes that the setting allows, of
// even length (ten steps, 5 and 5 against 7 and 3: L = 2048 77.9 us a trajectory
// against 83.2, L = 3000 130.7 and 138.3, L = 4096 216 and 221).
static int pass_steps(int n_md, int setting)
{
    const int most = std::min(std::min(setting, kMaxStepsPerPass), n_md), passes = (n_md + most - 1) / most;
    return (n_md + passes - 1) / passes;
}
constexpr int kPassWaves = 8;
constexpr int kPassFewRegions = 320;    // four rows a thread up to this many regions

template <int R>
__global__ void __launch_bounds__(kPassWaves * 64)
k_hmc_pass(const float* __restrict__ src, float* __restrict__ dst, const float* __restrict__ psrc,
           float* __restrict__ pdst, int L, int K, float kick0, float kick, float drift)
{
    __shared__ float4 lds[kPassLds<kPassWaves>];
    const int b = (int)xcd_band(blockIdx.x, gridDim.x);       // a grid of a multiple of 8
    if (b >= pass_tiles<kPassWaves, R>(L, K)) return;
    pass_body<kPassWaves, R>(src, dst, psrc, pdst, L, K, K, kick0, kick, drift, b, lds);
}

static void launch_pass(hipStream_t s, const float* src, float* dst, const float* psrc, float* pdst, int L, int k,
                        float kick0, float kick, float drift)
{
    const bool tall = pass_tiles<kPassWaves, 4>(L, k) > kPassFewRegions;
    const int nt = tall ? pass_tiles<kPassWaves, 8>(L, k) : pass_tiles<kPassWaves, 4>(L, k);
    const dim3 grid((unsigned)((nt + 7) & ~7)), block(kPassWaves * 64);
    if (tall)
        hipLaunchKernelGGL(k_hmc_pass<8>, grid, block, 0, s, src, dst, psrc, pdst, L, k, kick0, kick, drift);
    else
        hipLaunchKernelGGL(k_hmc_pass<4>, grid, block, 0, s, src, dst, psrc, pdst, L, k, kick0, kick, drift);
}

// Final half kick and the partial records of H_new; `copy` != NULL receives the
// angles (the final ones may sit in the second buffer).  Grid as k_hmc_begin.
__global__ void __launch_bounds__(kThreads)
k_hmc_end(const float* __restrict__ st, float* __restrict__ copy, const float* __restrict__ p, int L,
          float nbeta_kick, int cols, int rb, double* __restrict__ rec)
{
    const int Hh = L >> 1;
    const unsigned t = xcd_band(blockIdx.x, gridDim.x);
    const int col = (int)(t % (unsigned)cols);
    const int k = (col >> 1) * kThreads + threadIdx.x;
    const int c = col & 1;
    double v[7] = {0, 0, 0, 0, 0, 0, 0};
    const int R = (L + rb - 1) / rb, y0 = (int)(t / (unsigned)cols) * R, y1 = y0 + R < L ? y0 + R : L;
    if (k < Hh) {
        for (int y = y0; y < y1; ++y) {
            float th;
            const Nb n = load_nb(st, L, Hh, c, y, k, th);
            const size_t i = ((size_t)c * L + y) * Hh + k;
            if (copy) copy[i] = th;
            const float pn = __fmaf_rn(nbeta_kick, sin_sum(n), p[i]);
            accumulate(v, n, c, __fmul_rn(0.5f, __fmul_rn(pn, pn)));
        }
    }
    write_record(v, rec, t);
}

// Begin and end of a trajectory for L % 4 == 0, by pairs: a thread takes pair j
// (entries 2j, 2j+1) of both colours in a run of consecutive rows.  Each plane's
// pair j of the rows above, at and below a row sits in registers as a rolling
// window with its (cos, sin): a row loads one new pair of each plane and one edge
// entry of each (2j-1 or 2j+2), so every angle is read from memory once (a thread
// per colour would read each plane twice, once as its own colour and once as the
// other's neighbours) and a site costs 1.5 sines and cosines.
// 1-D grid of cols2 = ceil(J/256) column blocks times the row blocks, remapped by
// xcd_band; a row block holds ends_group(L) runs side by side (one unless
// J < 256); one partial record per wave.
struct PairCS {
    float c0, s0, c1, s1;
};
__device__ __forceinline__ PairCS pair_cs(float2 t)
{
    PairCS q;
    sincos_turn(t.x, q.s0, q.c0);
    sincos_turn(t.y, q.s1, q.c1);
    return q;
}

// Neighbourhoods of the pair (entries 2j, 2j+1) of row y: own (cos, sin) in a,
// b; the other plane's row above (u), at (h) and below (d) and the edge entry e.
__device__ __forceinline__ void pair_nb(const PairCS& own, const PairCS& u, const PairCS& h, const PairCS& d,
                                       float ce, float se, int o, Nb& na, Nb& nb)
{
    na.c = own.c0; na.s = own.s0;
    nb.c = own.c1; nb.s = own.s1;
    // entry 2j: left = (o ? h0 : e), right = (o ? h1 : h0); 2j+1: left = (o ? h1 : h0), right = (o ? e : h1)
    na.cl = o ? h.c0 : ce;   na.sl = o ? h.s0 : se;
    na.cr = o ? h.c1 : h.c0; na.sr = o ? h.s1 : h.s0;
    nb.cl = o ? h.c1 : h.c0; nb.sl = o ? h.s1 : h.s0;
    nb.cr = o ? ce : h.c1;   nb.sr = o ? se : h.s1;
    na.cu = u.c0; na.su = u.s0; nb.cu = u.c1; nb.su = u.s1;
    na.cd = d.c0; na.sd = d.s0; nb.cd = d.c1; nb.sd = d.s1;
}

// Pair columns per run and runs per workgroup of the pair kernels: a lattice
// narrower than a workgroup (J < 256 pair columns) gives each workgroup
// 256 / J runs side by side instead of leaving lanes idle.
__host__ __device__ __forceinline__ int ends_group(int L)
{
    const int J = L >> 2;
    return kThreads / (J < kThreads ? (J > 0 ? J : 1) : kThreads);
}

// The pass on record block t (after the XCD remap) of one lattice, whose rows
// are cut into `runs` runs of equal length (the last may be shorter).
template <bool BEGIN>
__device__ __forceinline__ void ends2_body(const float* __restrict__ st, float* __restrict__ p,
                                           float* __restrict__ copy, int L, uint32_t traj, uint32_t k0, uint32_t k1,
                                           float nbeta_kick, int cols, int runs, double* __restrict__ rec, unsigned t)
{
    const int Hh = L >> 1, J = Hh >> 1;
    const int G = ends_group(L), JB = kThreads / G;
    const int col = (int)(t % (unsigned)cols);
    const int g = (int)threadIdx.x / JB;
    const int j = col * kThreads + (int)threadIdx.x - g * JB;
    const int run = (int)(t / (unsigned)cols) * G + g;
    double v[7] = {0, 0, 0, 0, 0, 0, 0};
    const int R = (L + runs - 1) / runs, y0 = run * R, y1 = y0 + R < L ? y0 + R : L;
    if (g < G && j < J && y0 < y1) {
        const float* pl0 = st;
        const float* pl1 = st + (size_t)L * Hh;
        const float2* r0 = (const float2*)pl0;
        const float2* r1 = (const float2*)pl1;
        // windows: plane c rows y-1 (u), y (h) with angles, y+1 loaded per row
        float2 t0 = r0[(size_t)y0 * J + j], t1 = r1[(size_t)y0 * J + j];
        PairCS u0 = pair_cs(r0[(size_t)wrapi(y0 - 1, L) * J + j]), u1 = pair_cs(r1[(size_t)wrapi(y0 - 1, L) * J + j]);
        PairCS h0 = pair_cs(t0), h1 = pair_cs(t1);
        const int kl = wrapi(2 * j - 1, Hh), kr = wrapi(2 * j + 2, Hh);
        for (int y = y0; y < y1; ++y) {
            const int yd = wrapi(y + 1, L);
            const float2 n0 = r0[(size_t)yd * J + j], n1 = r1[(size_t)yd * J + j];
            const PairCS d0 = pair_cs(n0), d1 = pair_cs(n1);
            const int o = y & 1;                  // red rows: o = y & 1; black rows: 1 - o
            // edge entries: the red pair reads plane 1 at 2j+2 (o) or 2j-1; the black pair plane 0 the other way
            float se1, ce1, se0, ce0;
            sincos_turn(pl1[(size_t)y * Hh + (o ? kr : kl)], se1, ce1);
            sincos_turn(pl0[(size_t)y * Hh + (o ? kl : kr)], se0, ce0);
            Nb na0, nb0, na1, nb1;
            pair_nb(h0, u1, h1, d1, ce1, se1, o, na0, nb0);
            pair_nb(h1, u0, h0, d0, ce0, se0, 1 - o, na1, nb1);
            const size_t row0 = (size_t)y * Hh, row1 = ((size_t)L + y) * Hh;
            float pa0, pb0, pa1, pb1;
            if constexpr (BEGIN) {
                ((float2*)(copy + row0))[j] = t0;      // saved angles
                ((float2*)(copy + row1))[j] = t1;
                const u32x4 q0 = philox10(traj, 0u, 2u, (uint32_t)y * (uint32_t)J + (uint32_t)j, k0, k1);
                const u32x4 q1 = philox10(traj, 1u, 2u, (uint32_t)y * (uint32_t)J + (uint32_t)j, k0, k1);
                pa0 = box_muller(q0.x, q0.y);
                pb0 = box_muller(q0.z, q0.w);
                pa1 = box_muller(q1.x, q1.y);
                pb1 = box_muller(q1.z, q1.w);
                ((float2*)(p + row0))[j] = make_float2(pa0, pb0);
                ((float2*)(p + row1))[j] = make_float2(pa1, pb1);
            } else {
                if (copy) {
                    ((float2*)(copy + row0))[j] = t0;
                    ((float2*)(copy + row1))[j] = t1;
                }
                const float2 pv0 = ((const float2*)(p + row0))[j], pv1 = ((const float2*)(p + row1))[j];
                pa0 = __fmaf_rn(nbeta_kick, sin_sum(na0), pv0.x);
                pb0 = __fmaf_rn(nbeta_kick, sin_sum(nb0), pv0.y);
                pa1 = __fmaf_rn(nbeta_kick, sin_sum(na1), pv1.x);
                pb1 = __fmaf_rn(nbeta_kick, sin_sum(nb1), pv1.y);
            }
            accumulate(v, na0, 0, __fmul_rn(0.5f, __fmul_rn(pa0, pa0)));
            accumulate(v, nb0, 0, __fmul_rn(0.5f, __fmul_rn(pb0, pb0)));
            accumulate(v, na1, 1, __fmul_rn(0.5f, __fmul_rn(pa1, pa1)));
            accumulate(v, nb1, 1, __fmul_rn(0.5f, __fmul_rn(pb1, pb1)));
            u0 = h0; u1 = h1;
            h0 = d0; h1 = d1;
            t0 = n0; t1 = n1;
        }
    }
    write_record(v, rec, t);              // every lane reaches the wave sums
}

template <bool BEGIN>
__global__ void __launch_bounds__(kThreads)
k_hmc_ends2(float* st, float* __restrict__ p, float* copy, int L, uint32_t traj,
            uint32_t k0, uint32_t k1, float nbeta_kick, int cols, int rb, int again, unsigned* __restrict__ flag,
            double* __restrict__ rec)
{
    if (BEGIN && blockIdx.x == 0 && threadIdx.x == 0) flag[1] = 0u;
    const bool back = BEGIN && rejected_before(again, flag);
    ends2_body<BEGIN>(back ? copy : st, p, back ? st : copy, L, traj, k0, k1, nbeta_kick, cols, rb, rec, xcd_band(blockIdx.x, gridDim.x));
}

// Metropolis step of the trajectory.  Workgroup b sums chunk b % nchunk (256
// records) of the old records, or of the new ones from nchunk on; the one that
// arrives last (a counter behind the flag, zeroed by the begin kernel; released and
// acquired at device scope) sums the chunk results in their order and decides.
// Three launches of 2.8 us each otherwise.
__device__ __forceinline__ void decide_body(const double* __restrict__ rec_old, const double* __restrict__ rec_new,
                                            int nrec, int nchunk, double* __restrict__ chunk_old,
                                            double* __restrict__ chunk_new, double beta, uint32_t traj, uint32_t k0,
                                            uint32_t k1, unsigned* __restrict__ flag, xy_hmc_obs* __restrict__ obs)
{
    __shared__ double red[64], sums[16];
    __shared__ int last;
    const bool fresh = (int)blockIdx.x >= nchunk;
    const int ch = (int)blockIdx.x - (fresh ? nchunk : 0), i = ch * 256;
    const double s = column_sums((fresh ? rec_new : rec_old) + (size_t)i * 8, min(256, nrec - i), red);
    if (threadIdx.x < 8) {
        (fresh ? chunk_new : chunk_old)[(size_t)ch * 8 + threadIdx.x] = s;
        __threadfence();
        // lanes of one wave: the stores above are done before lane 0's arrival
        if (threadIdx.x == 0) last = atomicAdd(flag + 1, 1u) == gridDim.x - 1u;
    }
    __syncthreads();
    if (!last) return;
    __threadfence();
    const double o = column_sums(chunk_old, nchunk, red), n = column_sums(chunk_new, nchunk, red + 32);
    if (threadIdx.x < 8) {
        sums[threadIdx.x] = o;
        sums[8 + threadIdx.x] = n;
    }
    __syncthreads();
    if (threadIdx.x == 0) decide_core(sums, sums + 8, beta, traj, k0, k1, flag, obs);
}

__global__ void __launch_bounds__(kThreads)
k_hmc_decide(const double* __restrict__ rec_old, const double* __restrict__ rec_new, int nrec, int nchunk,
             double* __restrict__ chunk_old, double* __restrict__ chunk_new, double beta, uint32_t traj, uint32_t k0,
             uint32_t k1, unsigned* __restrict__ flag, xy_hmc_obs* __restrict__ obs)
{
    decide_body(rec_old, rec_new, nrec, nchunk, chunk_old, chunk_new, beta, traj, k0, k1, flag, obs);
}

// Rejected trajectory: the saved angles back into the state.
__global__ void __launch_bounds__(kThreads)
k_hmc_restore(const unsigned* __restrict__ flag, const float* __restrict__ saved, float* __restrict__ st, size_t n)
{
    if (*flag) return;
    for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (size_t)gridDim.x * kThreads)
        st[i] = saved[i];
}

// ----------------------------------------------------- four replicas of a quad
// The four lattices of a quad back to back (n floats each), taken by blockIdx.y:
// each stage is one launch of the single-lattice pass on all four.  Replica r's
// flag and arrival counter are flag[16 r], flag[16 r + 1].
__global__ void __launch_bounds__(kThreads)
k_quad_split(const float4* __restrict__ st, float* __restrict__ planes, size_t n)
{
    const size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const float4 v = st[i];
    planes[i] = v.x;
    planes[n + i] = v.y;
    planes[2 * n + i] = v.z;
    planes[3 * n + i] = v.w;
}

__global__ void __launch_bounds__(kThreads)
k_quad_join(const float* __restrict__ planes, float4* __restrict__ st, size_t n)
{
    const size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n) st[i] = make_float4(planes[i], planes[n + i], planes[2 * n + i], planes[3 * n + i]);
}

template <bool BEGIN>
__global__ void __launch_bounds__(kThreads)
k_qhmc_ends(float* st, float* __restrict__ p, float* copy, int L, uint32_t traj,
            QHmcKeys keys, float4 kick, int cols, int runs, int again, unsigned* __restrict__ flag,
            double* __restrict__ rec, int nrec)
{
    const int r = (int)blockIdx.y;
    const size_t o = (size_t)r * L * L;
    if (BEGIN && blockIdx.x == 0 && threadIdx.x == 0) flag[16 * r + 1] = 0u;
    float *from = st + o, *to = copy ? copy + o : nullptr;
    const bool back = BEGIN && rejected_before(again, flag + 16 * r);
    ends2_body<BEGIN>(back ? to : from, p + o, back ? from : to, L, traj, keys.k0[r], keys.k1[r],
                      r == 0 ? kick.x : r == 1 ? kick.y : r == 2 ? kick.z : kick.w, cols, runs,
                      rec + (size_t)r * nrec * 8, xcd_band(blockIdx.x, gridDim.x));
}

__global__ void __launch_bounds__(kThreads)
k_qhmc_step(const float* __restrict__ src, float* __restrict__ dst, float* __restrict__ p, int L, float4 kick,
            float drift)
{
    const int r = (int)blockIdx.y;
    const size_t o = (size_t)r * L * L;
    step2_body<kStepRows>(src + o, dst + o, p + o, L, r == 0 ? kick.x : r == 1 ? kick.y : r == 2 ? kick.z : kick.w,
                          drift, xcd_band(blockIdx.x, gridDim.x));
}

template <int R>
__global__ void __launch_bounds__(kPassWaves * 64)
k_qhmc_pass(const float* __restrict__ src, float* __restrict__ dst, const float* __restrict__ psrc,
            float* __restrict__ pdst, int L, int K, float4 kick0, float4 kick, float drift)
{
    __shared__ float4 lds[kPassLds<kPassWaves>];
    const int b = (int)xcd_band(blockIdx.x, gridDim.x), r = (int)blockIdx.y;
    if (b >= pass_tiles<kPassWaves, R>(L, K)) return;
    const size_t o = (size_t)r * L * L;
    const float ka = r == 0 ? kick0.x : r == 1 ? kick0.y : r == 2 ? kick0.z : kick0.w;
    const float kb = r == 0 ? kick.x : r == 1 ? kick.y : r == 2 ? kick.z : kick.w;
    pass_body<kPassWaves, R>(src + o, dst + o, psrc + o, pdst + o, L, K, K, ka, kb, drift, b, lds);
}

__global__ void __launch_bounds__(kThreads)
k_qhmc_decide(const double* __restrict__ rec_old, const double* __restrict__ rec_new, int nrec, int nchunk,
              double* __restrict__ chunk_old, double* __restrict__ chunk_new, QHmcBeta beta, uint32_t traj,
              QHmcKeys keys, unsigned* __restrict__ flag, xy_hmc_obs* __restrict__ obs)
{
    const int r = (int)blockIdx.y;
    const size_t o = (size_t)r * nrec * 8, c = (size_t)r * nchunk * 8;
    decide_body(rec_old + o, rec_new + o, nrec, nchunk, chunk_old + c, chunk_new + c, beta.b[r], traj, keys.k0[r],
                keys.k1[r], flag + 16 * r, obs ? obs + r : nullptr);
}

__global__ void __launch_bounds__(kThreads)
k_qhmc_restore(const unsigned* __restrict__ flag, const float* __restrict__ saved, float* __restrict__ st, size_t n)
{
    const int r = (int)blockIdx.y;
    if (flag[16 * r]) return;
    for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (size_t)gridDim.x * kThreads)
        st[r * n + i] = saved[r * n + i];
}

// ---------------------------------------------------------------- batches
// One launch per stage over all lattices of a batch.  A stage's grid is the
// lattices' single-lattice grids one after another, each padded to a multiple of
// 8 workgroups (so that each lattice's first workgroup goes to XCD 0 and the XCD
// remap gives it the same bands as alone); a workgroup finds its lattice by
// bisection over the stage's block offsets and runs the single-lattice pass on
// its local index.

// Lattice i with start[i] <= blk < start[i + 1].
__device__ __forceinline__ int bh_find(const uint32_t* __restrict__ start, int n, uint32_t blk)
{
    int lo = 0, hi = n;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (start[mid] <= blk) lo = mid;
        else hi = mid;
    }
    return lo;
}

// Trajectory ends: BEGIN draws the momenta, saves the angles and writes the H_old
// records; else the final half kick from the angles that the leap-frog passes left in
// the second buffer (parity odd, also copied back into the state) or the first, and
// the momenta (pparity) likewise, and the H_new records.
template <bool BEGIN>
__global__ void __launch_bounds__(kThreads)
k_bhmc_ends(const BhLat* __restrict__ d, const uint32_t* __restrict__ start, int n,
            const uint32_t* __restrict__ traj_dev, int parity, int pparity)
{
    const int i = bh_find(start, n, blockIdx.x);
    const BhLat& q = d[i];
    const int G = ends_group(q.L);
    const unsigned nb = (unsigned)(q.cols * ((q.rb + G - 1) / G)), lb = blockIdx.x - start[i];
    if (lb >= nb) return;
    const unsigned t = xcd_band(lb, nb);
    if constexpr (BEGIN)
        ends2_body<true>(q.st, q.w.p, q.w.saved, q.L, *traj_dev, q.k0, q.k1, 0.0f, q.cols, q.rb, q.w.rec_old, t);
    else
        ends2_body<false>(parity ? q.pp : q.st, pparity ? q.w.p2 : q.w.p, parity ? q.st : nullptr, q.L, 0u, q.k0,
                          q.k1, q.kick_half, q.cols, q.rb, q.w.rec_new, t);
}

// One leap-frog step of every lattice (L % 4 == 0), the momenta in place; parity odd:
// from the second angle buffer to the first.
__global__ void __launch_bounds__(kThreads)
k_bhmc_step(const BhLat* __restrict__ d, const uint32_t* __restrict__ start, int n, int parity, int first, float drift)
{
    const int i = bh_find(start, n, blockIdx.x);
    const BhLat& q = d[i];
    const unsigned t = xcd_band(blockIdx.x - start[i], start[i + 1] - start[i]);
    if (t >= step2_blocks(q.L)) return;
    step2_body<kStepRows>(parity ? q.pp : q.st, parity ? q.st : q.pp, q.w.p, q.L, first ? q.kick_half : q.kick_full,
                          drift, t);
}

// K leap-frog steps of every lattice, on regions cut for passes of KH; parity odd:
// the angles and momenta are read from the second buffers and written to the first.
template <int R>
__global__ void __launch_bounds__(kPassWaves * 64)
k_bhmc_pass(const BhLat* __restrict__ d, const uint32_t* __restrict__ start, int n, int KH, int K, int parity,
            int first, float drift)
{
    __shared__ float4 lds[kPassLds<kPassWaves>];
    const int i = bh_find(start, n, blockIdx.x);
    const BhLat& q = d[i];
    const unsigned lb = blockIdx.x - start[i];
    const int b = (int)xcd_band(lb, start[i + 1] - start[i]);
    if (b >= pass_tiles<kPassWaves, R>(q.L, KH)) return;
    pass_body<kPassWaves, R>(parity ? q.pp : q.st, parity ? q.st : q.pp, parity ? q.w.p2 : q.w.p,
                             parity ? q.w.p : q.w.p2, q.L, KH, K, first ? q.kick_half : q.kick_full, q.kick_full,
                             drift, b, lds);
}

// One lattice's records summed as the single-lattice trajectory sums them: chunks
// of 256 records (into ch, LDS), then the chunk sums.  Threads 0 .. 7 get their
// column's total.
__device__ double bh_sum(const double* __restrict__ rec, int nrec, double* ch, double* red)
{
    const int nch = (nrec + 255) / 256;
    for (int c = 0; c < nch; ++c) {
        const double s = column_sums(rec + (size_t)c * 256 * 8, min(256, nrec - c * 256), red + (c & 1) * 32);
        if (threadIdx.x < 8) ch[c * 8 + threadIdx.x] = s;
    }
    __syncthreads();
    return column_sums(ch, nch, red);
}

// Metropolis step of every lattice: workgroup i on lattice i.
__global__ void __launch_bounds__(kThreads)
k_bhmc_decide(const BhLat* __restrict__ d, const uint32_t* __restrict__ traj_dev)
{
    __shared__ double red[64], sums[16];
    __shared__ double ch[kHmcMaxChunks * 8];
    const BhLat& q = d[blockIdx.x];
    const double o = bh_sum(q.w.rec_old, q.nrec, ch, red);
    __syncthreads();
    const double n = bh_sum(q.w.rec_new, q.nrec, ch, red);
    if (threadIdx.x < 8) {
        sums[threadIdx.x] = o;
        sums[8 + threadIdx.x] = n;
    }
    __syncthreads();
    if (threadIdx.x == 0) decide_core(sums, sums + 8, q.beta, *traj_dev, q.k0, q.k1, q.w.flag, q.obs);
}

// Rejected trajectories: the saved angles back into the state.
__global__ void __launch_bounds__(kThreads)
k_bhmc_restore(const BhLat* __restrict__ d, const uint32_t* __restrict__ start, int n)
{
    const int i = bh_find(start, n, blockIdx.x);
    const BhLat& q = d[i];
    if (*q.w.flag) return;
    const size_t ns = (size_t)q.L * (size_t)q.L;
    const size_t stride = (size_t)(start[i + 1] - start[i]) * kThreads;
    for (size_t j = (size_t)(blockIdx.x - start[i]) * kThreads + threadIdx.x; j < ns; j += stride)
        q.st[j] = q.w.saved[j];
}

}  // namespace

// Block columns (both colours) and row blocks of the record-writing kernels: as
// many rows as keep one record set at most kHmcMaxRecords.
static int hmc_cols(int L) { return 2 * (((L >> 1) + kThreads - 1) / kThreads); }

static int hmc_row_blocks(int L)
{
    int gy = kHmcMaxRecords / (hmc_cols(L) * (kThreads / 64));
    if (gy > L) gy = L;
    return gy < 1 ? 1 : gy;
}

static bool hmc_pairs(int L) { return L % 4 == 0; }
static int hmc_cols2(int L) { return ((L >> 2) + kThreads - 1) / kThreads; }
// Row runs of the pair kernels.  Each run reads the plane rows just above and
// below it once more and starts its rolling window with their sines and
// cosines, so short runs cost traffic and arithmetic.  Lattices of more than one
// column block (L > 1024): runs of up to 32 rows, but at least about 2048
// workgroups while L allows, and at most one record per wave within the record
// buffer.  One column block (L <= 1024): runs of 8 rows where batches of many
// lattices supply the parallelism (runs of 4 cost the 96-lattice scan 1.8%), of 4 or
// 2 where a lattice is a few workgroups whose runs are one long chain (L = 256: 35 us
// a trajectory of 20 steps against 47).
static int hmc_runs2(int L, int max_records = kHmcMaxRecords)
{
    const int cols = hmc_cols2(L);
    if (cols == 1) return L <= 256 ? L / 2 : L <= 512 ? (L + 3) / 4 : (L + 7) / 8;
    int gy = (2048 + cols - 1) / cols;
    if (gy < L / 32) gy = L / 32;
    const int cap = max_records / (cols * (kThreads / 64));
    if (gy > cap) gy = cap;
    if (gy > L) gy = L;
    return gy < 1 ? 1 : gy;
}
// Workgroups per column block: the runs, ends_group(L) to a workgroup.
static int hmc_row_blocks2(int L)
{
    const int G = ends_group(L);
    return (hmc_runs2(L) + G - 1) / G;
}

int hmc_records(int L)
{
    if (hmc_pairs(L)) return hmc_cols2(L) * hmc_row_blocks2(L) * (kThreads / 64);
    return hmc_cols(L) * hmc_row_blocks(L) * (kThreads / 64);
}

size_t hmc_work_bytes(int L)
{
    const size_t n = (size_t)L * (size_t)L;
    return 256 + 3 * n * sizeof(float) + 2 * (size_t)(kHmcMaxRecords + kHmcMaxChunks) * 8 * sizeof(double);
}

HmcWork hmc_carve(void* work, int L)
{
    HmcWork w;
    char* b = (char*)work;
    w.flag = (unsigned*)b;
    b += 256;
    const size_t n = (size_t)L * (size_t)L;
    w.p = (float*)b;
    b += n * sizeof(float);
    w.saved = (float*)b;
    b += n * sizeof(float);
    w.p2 = (float*)b;
    b += n * sizeof(float);
    w.rec_old = (double*)b;
    b += (size_t)kHmcMaxRecords * 8 * sizeof(double);
    w.rec_new = (double*)b;
    b += (size_t)kHmcMaxRecords * 8 * sizeof(double);
    w.chunk_old = (double*)b;
    b += (size_t)kHmcMaxChunks * 8 * sizeof(double);
    w.chunk_new = (double*)b;
    return w;
}

// The same areas with the record arrays sized for this L only (batches).
size_t hmc_work_bytes_compact(int L)
{
    const size_t n = (size_t)L * (size_t)L;
    const size_t nrec = (size_t)hmc_records(L), nch = (nrec + 255) / 256;
    return 256 + 3 * n * sizeof(float) + 2 * (nrec + nch) * 8 * sizeof(double);
}

HmcWork hmc_carve_compact(void* work, int L)
{
    HmcWork w;
    char* b = (char*)work;
    const size_t n = (size_t)L * (size_t)L;
    const size_t nrec = (size_t)hmc_records(L), nch = (nrec + 255) / 256;
    w.flag = (unsigned*)b;
    b += 256;
    w.p = (float*)b;
    b += n * sizeof(float);
    w.saved = (float*)b;
    b += n * sizeof(float);
    w.p2 = (float*)b;
    b += n * sizeof(float);
    w.rec_old = (double*)b;
    b += nrec * 8 * sizeof(double);
    w.rec_new = (double*)b;
    b += nrec * 8 * sizeof(double);
    w.chunk_old = (double*)b;
    b += nch * 8 * sizeof(double);
    w.chunk_new = (double*)b;
    return w;
}

hipError_t launch_hmc_trajectory(float* state, float* pingpong, const HmcWork& w, int L, double beta, double eps,
                                 int n_md, int steps_per_pass, uint32_t traj, uint32_t k0, uint32_t k1,
                                 xy_hmc_obs* obs, bool again, hipStream_t s)
{
    const bool pairs2 = hmc_pairs(L);
    const int cols = pairs2 ? hmc_cols2(L) : hmc_cols(L), rb = pairs2 ? hmc_runs2(L) : hmc_row_blocks(L);
    const int nbr = pairs2 ? hmc_row_blocks2(L) : rb;     // workgroups per column block
    const dim3 grec((unsigned)(cols * nbr)), gstep(hmc_cols(L), L), block(kThreads);
    const int nrec = hmc_records(L);
    const int nchunk = (nrec + 255) / 256;
    const float drift = (float)(eps / (2.0 * 3.14159265358979323846));
    if (pairs2)
        hipLaunchKernelGGL(k_hmc_ends2<true>, grec, block, 0, s, state, w.p, w.saved, L, traj, k0, k1, 0.0f, cols, rb,
                           (int)again, w.flag, w.rec_old);
    else
        hipLaunchKernelGGL(k_hmc_begin, grec, block, 0, s, state, w.p, w.saved, L, traj, k0, k1, cols, rb,
                           (int)again, w.flag, w.rec_old);
    float* src = state;
    float* dst = pingpong;
    float* p = w.p;
    const float kick_half = (float)(-beta * 0.5 * eps), kick_full = (float)(-beta * eps);
    if (steps_per_pass > 1) {
        // passes of up to steps_per_pass steps; the momenta ping-pong between p and p2
        float* pn = w.p2;
        const int kmax = pass_steps(n_md, steps_per_pass);
        for (int q = 0; q < n_md;) {
            const int k = n_md - q < kmax ? n_md - q : kmax;
            launch_pass(s, src, dst, p, pn, L, k, q == 0 ? kick_half : kick_full, kick_full, drift);
            float* t = src;
            src = dst;
            dst = t;
            t = p;
            p = pn;
            pn = t;
            q += k;
        }
    } else {
        const bool pairs = (L % (4 * kStepRows)) == 0;
        for (int q = 0; q < n_md; ++q) {
            const float kick = q == 0 ? kick_half : kick_full;
            if (pairs)
                hipLaunchKernelGGL(k_hmc_step2, dim3(step2_blocks(L)), block, 0, s, src, dst, p, L, kick, drift);
            else
                hipLaunchKernelGGL(k_hmc_step, gstep, block, 0, s, src, dst, p, L, kick, drift);
            float* t = src;
            src = dst;
            dst = t;
        }
    }
    if (pairs2)
        hipLaunchKernelGGL(k_hmc_ends2<false>, grec, block, 0, s, src, p, src == state ? nullptr : state, L, traj, k0,
                           k1, kick_half, cols, rb, 0, w.flag, w.rec_new);
    else
        hipLaunchKernelGGL(k_hmc_end, grec, block, 0, s, src, src == state ? nullptr : state, p, L, kick_half, cols,
                           rb, w.rec_new);
    hipLaunchKernelGGL(k_hmc_decide, dim3(2 * (unsigned)nchunk), block, 0, s, w.rec_old, w.rec_new, nrec, nchunk,
                       w.chunk_old, w.chunk_new, beta, traj, k0, k1, w.flag, obs);
    return hipGetLastError();
}

hipError_t launch_hmc_restore(float* state, const HmcWork& w, int L, hipStream_t s)
{
    const size_t n = (size_t)L * (size_t)L;
    const unsigned nb = (unsigned)((n + kThreads * 8 - 1) / (kThreads * 8));
    hipLaunchKernelGGL(k_hmc_restore, dim3(nb < 4096 ? nb : 4096), dim3(kThreads), 0, s, w.flag, w.saved, state, n);
    return hipGetLastError();
}

void hmc_batch_describe(BhLat& d, int L, double beta, double eps)
{
    d.L = L;
    d.beta = beta;
    d.cols = hmc_cols2(L);
    d.rb = hmc_runs2(L);
    d.nrec = hmc_records(L);
    d.kick_half = (float)(-beta * 0.5 * eps);
    d.kick_full = (float)(-beta * eps);
}

static uint32_t pad8(uint32_t v) { return (v + 7u) & ~7u; }

int hmc_batch_steps(int n_md, int steps_per_pass) { return pass_steps(n_md, steps_per_pass); }

int hmc_batch_rows(int n, const int32_t* L, int kh)
{
    // one step a pass: a region's halo, and momenta that move to another buffer, are not
    // worth it (four lattices of L = 2048, 20 steps: 2589 us a trajectory in regions, 1816)
    if (kh == 1) return 0;
    long long tiles = 0;
    for (int i = 0; i < n; ++i) tiles += pass_tiles<kPassWaves, 4>(L[i], kh);
    return tiles > kPassFewRegions ? 8 : 4;
}

void hmc_batch_blocks(int L, int rows, int kh, uint32_t nb[3])
{
    nb[0] = pad8((uint32_t)(hmc_cols2(L) * hmc_row_blocks2(L)));
    nb[1] = pad8((uint32_t)(rows == 0 ? step2_blocks(L) : rows == 8 ? pass_tiles<kPassWaves, 8>(L, kh) : pass_tiles<kPassWaves, 4>(L, kh)));
    const size_t n = (size_t)L * (size_t)L;
    const size_t r = (n + kThreads * 8 - 1) / (kThreads * 8);
    nb[2] = pad8((uint32_t)(r < 4096 ? r : 4096));
}

hipError_t launch_hmc_batch_trajectory(const BhLat* d, const uint32_t* start, int n, const uint32_t totals[3],
                                       double eps, int n_md, int steps_per_pass, int rows, const uint32_t* traj_dev,
                                       hipStream_t s)
{
    const uint32_t* s_ends = start;
    const uint32_t* s_pass = start + (n + 1);
    const uint32_t* s_rest = start + 2 * (n + 1);
    const float drift = (float)(eps / (2.0 * 3.14159265358979323846));
    const dim3 block(kThreads);
    hipLaunchKernelGGL(k_bhmc_ends<true>, dim3(totals[0]), block, 0, s, d, s_ends, n, traj_dev, 0, 0);
    const int kh = hmc_batch_steps(n_md, steps_per_pass);
    const dim3 bpass(kPassWaves * 64);
    int parity = 0;
    for (int q = 0; q < n_md;) {
        const int k = n_md - q < kh ? n_md - q : kh;
        if (rows == 0)
            hipLaunchKernelGGL(k_bhmc_step, dim3(totals[1]), block, 0, s, d, s_pass, n, parity, q == 0, drift);
        else if (rows == 8)
            hipLaunchKernelGGL(k_bhmc_pass<8>, dim3(totals[1]), bpass, 0, s, d, s_pass, n, kh, k, parity, q == 0, drift);
        else
            hipLaunchKernelGGL(k_bhmc_pass<4>, dim3(totals[1]), bpass, 0, s, d, s_pass, n, kh, k, parity, q == 0, drift);
        parity ^= 1;
        q += k;
    }
    hipLaunchKernelGGL(k_bhmc_ends<false>, dim3(totals[0]), block, 0, s, d, s_ends, n, traj_dev, parity,
                       rows == 0 ? 0 : parity);
    hipLaunchKernelGGL(k_bhmc_decide, dim3((unsigned)n), block, 0, s, d, traj_dev);
    hipLaunchKernelGGL(k_bhmc_restore, dim3(totals[2]), block, 0, s, d, s_rest, n);
    return hipGetLastError();
}

// ----------------------------------------------------- four replicas of a quad
// Partial records a quad's workspace holds per replica and H sum.
int quad_hmc_records(int L)
{
    const int cols = 2 * (((L >> 1) + kThreads - 1) / kThreads), rb = 4096 / cols;
    return cols * (rb < L ? (rb > 0 ? rb : 1) : L) * (kThreads / 64);
}

size_t quad_hmc_work_bytes(int L)
{
    const size_t st = ((size_t)L * L * sizeof(float4) + 255) & ~(size_t)255;
    const size_t nrec = (size_t)quad_hmc_records(L), nch = (nrec + 255) / 256;
    return 3 * st + 256 + 2 * 4 * (nrec + nch) * 8 * sizeof(double);
}

QuadHmcWork quad_hmc_carve(void* work, int L)
{
    const size_t st = ((size_t)L * L * sizeof(float4) + 255) & ~(size_t)255;
    const size_t nrec = (size_t)quad_hmc_records(L), nch = (nrec + 255) / 256;
    char* b = (char*)work;
    QuadHmcWork w;
    w.p = (float*)b;
    b += st;
    w.saved = (float*)b;
    b += st;
    w.p2 = (float*)b;
    b += st;
    w.flag = (unsigned*)b;
    b += 256;
    w.rec_old = (double*)b;
    b += 4 * nrec * 8 * sizeof(double);
    w.rec_new = (double*)b;
    b += 4 * nrec * 8 * sizeof(double);
    w.chunk_old = (double*)b;
    b += 4 * nch * 8 * sizeof(double);
    w.chunk_new = (double*)b;
    return w;
}

hipError_t launch_quad_split(const float4* state, float* planes, int L, hipStream_t s)
{
    const size_t n = (size_t)L * L;
    hipLaunchKernelGGL(k_quad_split, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, s, state,
                       planes, n);
    return hipGetLastError();
}

hipError_t launch_quad_join(const float* planes, float4* state, int L, hipStream_t s)
{
    const size_t n = (size_t)L * L;
    hipLaunchKernelGGL(k_quad_join, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, s, planes,
                       state, n);
    return hipGetLastError();
}

hipError_t launch_quad_hmc_trajectory(float* planes, float* second, const QuadHmcWork& w, int L, const double beta[4],
                                      double eps, int n_md, int steps_per_pass, uint32_t traj, const QHmcKeys& keys,
                                      xy_hmc_obs* obs, bool again, hipStream_t s)
{
    const int cols = hmc_cols2(L), runs = hmc_runs2(L, quad_hmc_records(L));
    const int G = ends_group(L), nbr = (runs + G - 1) / G;
    const int nrec = cols * nbr * (kThreads / 64), nchunk = (nrec + 255) / 256;
    const dim3 grec((unsigned)(cols * nbr), 4), block(kThreads), bpass(kPassWaves * 64);
    // the single-lattice launcher's FP32 constants, per replica
    const float drift = (float)(eps / (2.0 * 3.14159265358979323846));
    float kh[4], kf[4];
    QHmcBeta qb;
    for (int r = 0; r < 4; ++r) {
        kh[r] = (float)(-beta[r] * 0.5 * eps);
        kf[r] = (float)(-beta[r] * eps);
        qb.b[r] = beta[r];
    }
    const float4 kick_half = make_float4(kh[0], kh[1], kh[2], kh[3]);
    const float4 kick_full = make_float4(kf[0], kf[1], kf[2], kf[3]);
    hipLaunchKernelGGL(k_qhmc_ends<true>, grec, block, 0, s, planes, w.p, w.saved, L, traj, keys, kick_half, cols, runs,
                       (int)again, w.flag, w.rec_old, nrec);
    float *src = planes, *dst = second, *p = w.p, *pn = w.p2;
    const int kmax = pass_steps(n_md, steps_per_pass);
    for (int q = 0; q < n_md;) {
        const int k = std::min(n_md - q, kmax);
        const float4 k0 = q == 0 ? kick_half : kick_full;
        if (kmax == 1) {
            hipLaunchKernelGGL(k_qhmc_step, dim3(step2_blocks(L), 4), block, 0, s, src, dst, p, L, k0, drift);
            std::swap(src, dst);
            ++q;
            continue;
        }
        const bool tall = 4 * pass_tiles<kPassWaves, 4>(L, k) > kPassFewRegions;
        const int nt = tall ? pass_tiles<kPassWaves, 8>(L, k) : pass_tiles<kPassWaves, 4>(L, k);
        const dim3 grid((unsigned)((nt + 7) & ~7), 4);
        if (tall)
            hipLaunchKernelGGL(k_qhmc_pass<8>, grid, bpass, 0, s, src, dst, p, pn, L, k, k0, kick_full, drift);
        else
            hipLaunchKernelGGL(k_qhmc_pass<4>, grid, bpass, 0, s, src, dst, p, pn, L, k, k0, kick_full, drift);
        std::swap(src, dst);
        std::swap(p, pn);
        q += k;
    }
    hipLaunchKernelGGL(k_qhmc_ends<false>, grec, block, 0, s, src, p, src == planes ? nullptr : planes, L, traj, keys,
                       kick_half, cols, runs, 0, w.flag, w.rec_new, nrec);
    hipLaunchKernelGGL(k_qhmc_decide, dim3(2 * (unsigned)nchunk, 4), block, 0, s, w.rec_old, w.rec_new, nrec, nchunk,
                       w.chunk_old, w.chunk_new, qb, traj, keys, w.flag, obs);
    return hipGetLastError();
}

hipError_t launch_quad_hmc_restore(float* planes, const QuadHmcWork& w, int L, hipStream_t s)
{
    const size_t n = (size_t)L * (size_t)L;
    const unsigned nb = (unsigned)((n + kThreads * 8 - 1) / (kThreads * 8));
    hipLaunchKernelGGL(k_qhmc_restore, dim3(nb < 2048 ? nb : 2048, 4), dim3(kThreads), 0, s, w.flag, w.saved, planes, n);
    return hipGetLastError();
}

}  // namespace xyk
