// xy_deep.hip -- several sweeps of a single lattice per launch: one workgroup per
// region of xy_deep.hpp (the lattices too large for one workgroup and too small
// to keep the device busy for much longer than a launch takes).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "xy_deep.hpp"
#include "xy_launch.hpp"
#include "xy_reduce.hpp"

using namespace xyd;

namespace xyk {

// The lattice's pairs and rows are cut into tx x ty cores whose sides differ by
// at most one.
template <typename T, int NT, int R, bool ODD, int MEAS>
__global__ void __launch_bounds__(NT)
k_deep(const T* __restrict__ src, T* __restrict__ dst, int L, int tx, int ty, int PC, int RY, int hx, int hy,
       uint32_t sweep0, int n, int me, int phase, int rp, int full, uint32_t k0, uint32_t k1, Params p,
       double* __restrict__ part)
{
    extern __shared__ __align__(16) char smem[];
    const int nb = (int)gridDim.x, b = (int)blockIdx.x;
    const int by = b / tx, bx = b - by * tx;
    DeepRegion g;
    g.L = L;
    g.Hh = L >> 1;
    g.P = (g.Hh + 1) >> 1;
    const int c0 = (int)((long long)bx * g.P / tx), c1 = (int)((long long)(bx + 1) * g.P / tx);
    const int r0 = (int)((long long)by * L / ty), r1 = (int)((long long)(by + 1) * L / ty);
    g.ps = c0 - hx < 0 ? c0 - hx + g.P : c0 - hx;
    g.ys = r0 - hy < 0 ? r0 - hy + L : r0 - hy;
    g.PC = PC;
    g.RY = RY;
    g.hx = hx;
    g.hy = hy;
    g.cp = c1 - c0;
    g.cr = r1 - r0;
    deep_program<T, NT, R, ODD, false, MEAS>(src, dst, g, sweep0, n, me, phase, rp, full, k0, k1, p, smem,
                                             [&](int k, double s) { part[((size_t)k * nb + b) * 8 + threadIdx.x] = s; });
}

// Which lattices take several sweeps per launch, and into how many regions they
// are cut.  A launch costs about 3 us however little it does, and a half-sweep
// about 0.12 us plus 0.22 us for every wave that a SIMD has to run for it, so a
// region is the share of one CU: 16 x 16 regions, or regions of 16 x 16 sites
// where L <= 256, and as many sweeps as fit into the smallest workgroup that takes
// at least four.  Measured, us a sweep over long calls: L = 256 1.40 (single-sweep
// 256 x 16 tiles 4.84), L = 512 2.06 (4.97), L = 768 2.97 (5.13).  Below kDeepMinL
// the whole lattice in one workgroup is faster (L = 48: 1.6 against 2.0), beyond
// kDeepMaxL the halo's updates cost what the launches save (L = 1024: 4.4 over
// long calls, 5.5 over ten sweeps, against 5.0 for 128 x 16 tiles).
constexpr int kDeepMinL = 56, kDeepMaxL = 832, kDeepMaxSweeps = 8;

bool deep_region(int L, int n, DeepPlan* d)
{
    const int P = (L / 2 + 1) / 2;
    if (d->tx < 1 || d->ty < 1 || d->tx > P || d->ty > L || n < 1) return false;
    // halo: n entries of a half-row and 2 n rows; a region across the edge of an
    // L % 4 == 2 lattice holds one entry less
    d->hx = (n + (L % 4 ? 1 : 0) + 1) / 2;
    d->hy = 2 * n;
    d->PC = (P + d->tx - 1) / d->tx + 2 * d->hx;
    d->RY = ((L + d->ty - 1) / d->ty + 2 * d->hy + 1) & ~1;
    return d->PC <= P && d->RY <= L;
}

template <int NT, int R>
static bool deep_fits(const DeepPlan& d)
{
    return d.RY / 2 * d.PC <= kDeepPairs<NT, R> && deep_lds_bytes(d.PC, d.RY, NT) <= 160 * 1024;
}

bool deep_choose(int L, bool meas, DeepPlan* d, int* nmax)
{
    if (L < kDeepMinL || L > kDeepMaxL || L % 2) return false;
    d->tx = d->ty = std::min(16, (L + 15) / 16);
    d->rp = d->full = 0;
    if (meas && L % 64 == 0) {
        // the columns of the tile xy_get_plan reports: 256 x 16 (16 rows: four pairs,
        // 4 rows apart), 128 x 32 (32 rows: four, 8 apart), 64 x 32 (32 rows: two, 16
        // apart).  Cores of whole blocks of rows, their width again for one region a CU.
        d->rp = L % 256 == 0 ? 4 : L % 128 == 0 ? 8 : 16;
        d->full = L % 128 == 0 ? 4 : 2;
        if (L % 256 != 0) {
            const int P = L / 4;
            d->ty = L / 32;
            d->tx = std::min(P / 2, std::max(8192 / L, (P + 11) / 12));
        }
    }
    auto depth = [&](auto fits) {
        int n = kDeepMaxSweeps;
        while (n > 0 && !(deep_region(L, n, d) && fits(*d))) --n;
        return n;
    };
    int n = depth(deep_fits<512, 1>);
    if (n < 4) n = depth(deep_fits<1024, 1>);
    if (n < 4) n = depth(deep_fits<1024, 2>);
    *nmax = n;
    return n > 0;
}

template <typename T, int NT, int R, bool ODD, int MEAS>
static hipError_t run_deep(const SweepArgs& a, const DeepPlan& d, int n, int me, int phase, double* part,
                           hipStream_t s)
{
    static bool attr_set = false;
    auto kern = k_deep<T, NT, R, ODD, MEAS>;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const Params p{a.delta, a.nbl2e};
    hipLaunchKernelGGL(kern, dim3(d.tx * d.ty), dim3(NT), deep_lds_bytes(d.PC, d.RY, NT), s, (const T*)a.src,
                       (T*)a.dst, a.L, d.tx, d.ty, d.PC, d.RY, d.hx, d.hy, a.sweep, n, me, phase, d.rp,
                       d.full, a.key0, a.key1, p, part);
    return hipGetLastError();
}

template <typename T, bool ODD, int MEAS>
static hipError_t pick_deep(const SweepArgs& a, const DeepPlan& d, int n, int me, int phase, double* part,
                            hipStream_t s)
{
#define XY_DEEP(nt, r) \
    if (deep_fits<nt, r>(d)) return run_deep<T, nt, r, ODD, MEAS>(a, d, n, me, phase, part, s)
    XY_DEEP(512, 1);
    XY_DEEP(1024, 1);
    XY_DEEP(1024, 2);
#undef XY_DEEP
    return hipErrorInvalidValue;
}

template <typename T>
static hipError_t go_deep(const SweepArgs& a, const DeepPlan& d, int n, int me, int phase, double* part, hipStream_t s)
{
    const bool meas = me > 0 && (n + phase) / me > phase / me;
    if (a.L % 4)
        return meas ? pick_deep<T, true, kMeasPair>(a, d, n, me, phase, part, s)
                    : pick_deep<T, true, kMeasNone>(a, d, n, me, phase, part, s);
    if (meas && d.full) return pick_deep<T, false, kMeasChain>(a, d, n, me, phase, part, s);
    return meas ? pick_deep<T, false, kMeasPair>(a, d, n, me, phase, part, s)
                : pick_deep<T, false, kMeasNone>(a, d, n, me, phase, part, s);
}

hipError_t launch_deep(const SweepArgs& a, const DeepPlan& d, int n, int me, int phase, double* part, hipStream_t s)
{
    return a.precision == XY_FP16 ? go_deep<__half>(a, d, n, me, phase, part, s)
                                  : go_deep<float>(a, d, n, me, phase, part, s);
}

// Workgroup k: record k from its np partial records (fixed order), sweep count
// first + k * every.
__global__ void __launch_bounds__(256)
k_finalize_many(const double* __restrict__ part, int np, xy_obs* __restrict__ out, uint64_t first, int every)
{
    __shared__ double red[4 * 7];
    const int k = (int)blockIdx.x;
    double v[7] = {0, 0, 0, 0, 0, 0, 0};
    for (int i = threadIdx.x; i < np; i += 256) {
        const double* q = part + ((size_t)k * np + i) * 8;
#pragma unroll
        for (int c = 0; c < 7; ++c) v[c] += q[c];
    }
    block_sum7_256(v, red);
    if (threadIdx.x == 0) {
        xy_obs o;
        o.sweep = first + (uint64_t)k * (uint64_t)every;
        o.n_accept = (unsigned long long)v[6];
        o.cx = v[0]; o.cy = v[1]; o.ix = v[2]; o.iy = v[3]; o.mx = v[4]; o.my = v[5];
        out[k] = o;
    }
}

hipError_t launch_finalize_many(const double* part, int np, int nrec, xy_obs* out, uint64_t first, int every,
                                hipStream_t s)
{
    hipLaunchKernelGGL(k_finalize_many, dim3(nrec), dim3(256), 0, s, part, np, out, first, every);
    return hipGetLastError();
}

}  // namespace xyk
