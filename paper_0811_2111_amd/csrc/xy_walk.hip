// xy_walk.hip -- one sweep of large FP32 lattices by strips of one wave each
// (xy_walk.hpp), for a single lattice and for the four lattices of a quad.
#include <hip/hip_runtime.h>

#include "xy_launch.hpp"
#include "xy_tile4.hpp"
#include "xy_walk.hpp"

using namespace xyd;

namespace xyk {

// Wave w of the launch: strip w % strips of the run of rows w / strips, the runs as
// equal as even lengths can be; each XCD takes a band of runs.
template <bool MEAS, bool ST>
__device__ __forceinline__ void walk_block(const float* __restrict__ src, float* __restrict__ dst, int L, int runs,
                                           uint32_t sweep, uint32_t k0, uint32_t k1, const Params& p,
                                           double* __restrict__ part)
{
    const int strips = walk_strips(L);
    const int b = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);   // a multiple of 8
    const int w = b * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (w >= strips * runs) return;
    const int run = w / strips, s = w - run * strips;
    const int y0 = 2 * (int)((long long)run * (L >> 1) / runs), y1 = 2 * (int)((long long)(run + 1) * (L >> 1) / runs);
    walk_program<MEAS, ST>(src, dst, L, s, y0, y1 - y0, sweep, k0, k1, p, part + (size_t)w * 8);
}

template <bool MEAS, bool ST>
__global__ void __launch_bounds__(256)
k_walk(const float* __restrict__ src, float* __restrict__ dst, int L, int runs, uint32_t sweep, uint32_t k0,
       uint32_t k1, Params p, double* __restrict__ part)
{
    walk_block<MEAS, ST>(src, dst, L, runs, sweep, k0, k1, p, part);
}

// Replica blockIdx.y of four lattices back to back.
template <bool ST>
__global__ void __launch_bounds__(256)
k_walk_quad(const float* __restrict__ src, float* __restrict__ dst, int L, int runs, uint32_t sweep, Params4 p)
{
    const int r = (int)blockIdx.y;
    const size_t n = (size_t)r * L * L;
    const Params pr{p.delta[r], p.nbl2e[r]};
    walk_block<false, ST>(src + n, dst + n, L, runs, sweep, p.k0[r], p.k1[r], pr, nullptr);
}

// Lattices that sweep faster this way than by 256 x 16 tiles (us a sweep, tiles
// against this: L = 3072 18.6 and 19.2, 3584 25.2 and 24.8, 4096 30.7 and 29.7, 4608
// 39.0 and 37.4, 6000 71.4 and 66.1, 7000 94.5 and 86.1, 9600 171 and 165, 10000 196
// and 205) or by 512 x 64 strips of a workgroup (6144 77.1 and 67.5, 8192 119 and
// 113, 9216 153 and 162).  Below, the waves are too few; above, their rows, which
// share cache lines with the strips beside, cost the HBM more than the arithmetic
// saves.  FP16 gains nothing (L = 4096 29.1 and 32.3).
constexpr int kWalkMinL = 3500, kWalkMaxL = 9600, kWalkMaxStripL = 8192;

// Runs of about 16 rows: two more are updated a run, so longer ones do less work, but
// a SIMD needs several waves to fill its issue slots; as many as make the waves a
// multiple of the 1024 SIMDs (L = 4096: 300 runs of 13.6 rows, five waves a SIMD,
// 29.6 us; 240 of 17, four waves, 30.3; 256 of 16 32.2).
static int walk_runs(int L, int lattices)
{
    const int strips = walk_strips(L) * lattices;
    return 1024 * ((strips * (L / 16) + 1023) / 1024) / strips;
}

bool walk_supported(int L, int precision, bool meas)
{
    // a measured sweep by whole tiles is the faster one for 256 x 16 (L = 4096: 38.9 us
    // against 40.2 with FP32 chains of three rows) and, while the lattice is small, for 128 x 32 (tiles and strips: L =
    // 4224 44.8 and 47.2, 7040 113.3 and 113.4, 7296 122 and 119, 9600 212 and 203); not
    // for 64 x 32 (4160 48.8 and 43.1, 6080 97.4 and 86.5) or tiles cut off at the edge
    // (7000 119 and 114)
    const bool tiles = L % 256 == 0 || (L % 128 == 0 && L < 7200);
    return precision == XY_FP32 && L % 4 == 0 && L >= kWalkMinL && L <= (L % 512 ? kWalkMaxL : kWalkMaxStripL) &&
           !(meas && tiles);
}

int walk_records(int L) { return walk_strips(L) * walk_runs(L, 1); }

template <bool MEAS, bool ST>
static hipError_t run_walk(const SweepArgs& a, double* part, hipStream_t s)
{
    const int runs = walk_runs(a.L, 1);
    const unsigned nb = (unsigned)(walk_strips(a.L) * runs + 3) / 4;
    const Params p{a.delta, a.nbl2e};
    hipLaunchKernelGGL((k_walk<MEAS, ST>), dim3((nb + 7) & ~7u), dim3(256), 0, s, (const float*)a.src, (float*)a.dst,
                       a.L, runs, a.sweep, a.key0, a.key1, p, part);
    return hipGetLastError();
}

hipError_t launch_walk(const SweepArgs& a, bool meas, double* part, hipStream_t s)
{
    if (!walk_supported(a.L, a.precision, meas)) return hipErrorInvalidValue;
    const bool st = 2 * (size_t)a.L * (size_t)a.L * sizeof(float) > (size_t)256 << 20;
    if (meas) return st ? run_walk<true, true>(a, part, s) : run_walk<true, false>(a, part, s);
    return st ? run_walk<false, true>(a, part, s) : run_walk<false, false>(a, part, s);
}

// us a sweep of four lattices, by 256 x 16 tiles and this: L = 2528 45.6 and 45.9,
// 2816 56.2 and 52.6, 3584 93.0 and 90.3, 4096 123.5 and 115.1.
bool walk_quad_supported(int L) { return L % 4 == 0 && L >= 2800 && L <= 4608; }

hipError_t launch_walk_quad(const float* src, float* dst, int L, uint32_t sweep, const Params4& p, hipStream_t s)
{
    if (!walk_quad_supported(L)) return hipErrorInvalidValue;
    const int runs = walk_runs(L, 4);
    const dim3 grid(((unsigned)(walk_strips(L) * runs + 3) / 4 + 7) & ~7u, 4);
    if (2 * (size_t)L * (size_t)L * sizeof(float4) > (size_t)256 << 20)
        hipLaunchKernelGGL((k_walk_quad<true>), grid, dim3(256), 0, s, src, dst, L, runs, sweep, p);
    else
        hipLaunchKernelGGL((k_walk_quad<false>), grid, dim3(256), 0, s, src, dst, L, runs, sweep, p);
    return hipGetLastError();
}

}  // namespace xyk
