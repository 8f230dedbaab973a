// xy_deep.hip -- several sweeps of a single lattice per launch: one workgroup per
// region of xy_deep.hpp (the lattices too large for one workgroup and too small
// to keep the device busy for much longer than a launch takes).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "xy_deep.hpp"
#include "xy_launch.hpp"
#include "xy_reduce.hpp"
#include "xy_tile4.hpp"

using namespace xyd;

namespace xyk {

// The lattice's pairs and rows are cut into tx x ty cores whose sides differ by
// at most one.
__device__ __forceinline__ DeepRegion region_of(int b, int L, int tx, int ty, int PC, int RY, int hx, int hy)
{
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
    return g;
}

template <typename T, int NT, int R, bool ODD, int MEAS>
__global__ void __launch_bounds__(NT)
k_deep(const T* __restrict__ src, T* __restrict__ dst, int L, int tx, int ty, int PC, int RY, int hx, int hy,
       uint32_t sweep0, int n, int me, int phase, int rp, int full, uint32_t k0, uint32_t k1, Params p,
       double* __restrict__ part)
{
    extern __shared__ __align__(16) char smem[];
    const int nb = (int)gridDim.x, b = (int)blockIdx.x;
    const DeepRegion g = region_of(b, L, tx, ty, PC, RY, hx, hy);
    deep_program<T, NT, R, ODD, false, MEAS, false>(src, dst, g, sweep0, n, me, phase, rp, full, k0, k1, p, smem,
                                             [&](int k, double s) { part[((size_t)k * nb + b) * 8 + threadIdx.x] = s; });
}

// Which lattices take several sweeps per launch, and into how many regions they
// are cut.  A launch costs about 3 us however little it does, and a half-sweep
// about 0.12 us plus 0.22 us for every wave that a SIMD has to run for it, so a
// region is the share of one CU: 16 x 16 regions, or regions of 16 x 16 sites
// where L <= 256, and as many sweeps as fit into the smallest workgroup that takes
// at least four.  Measured, us a sweep over long calls: L = 256 1.40 (single-sweep
// 256 x 16 tiles 4.84), L = 512 2.06 (4.97), L = 768 2.97 (5.13), L = 832 3.4 (4.9,
// and 4.5 with two pairs a thread, which leave room for two sweeps a launch), L = 1024
// 4.1 (4.9).  Below kDeepMinL the whole lattice in one workgroup is faster (L = 48:
// 1.6 against 2.0), beyond kDeepMaxL the halo's updates cost what the launches save
// (ten sweeps: L = 1000 4.3 against 5.0 for 128 x 16 tiles, L = 1088 4.5 and 5.7, L =
// 1200 6.0 and 5.9, L = 1280 7.8 and 6.5).
constexpr int kDeepMinL = 56, kDeepMaxL = 1100, kDeepMaxSweeps = 8;

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

// The most sweeps of d's cores in the smallest workgroup that takes at least four.
static int deep_depth(int L, DeepPlan* d)
{
    auto depth = [&](auto fits) {
        int n = kDeepMaxSweeps;
        while (n > 0 && !(deep_region(L, n, d) && fits(*d))) --n;
        return n;
    };
    int n = depth(deep_fits<512, 1>);
    if (n < 4) n = depth(deep_fits<1024, 1>);
    if (n < 4) n = depth(deep_fits<1024, 2>);
    if (n < 4) n = depth(deep_fits<1024, 4>);
    return n;
}

bool deep_choose(int L, int64_t n, bool meas, DeepPlan* d, int* nmax)
{
    // a single sweep gains nothing, nor do two from L = 384 on (8.5 us against 7.8 by
    // tiles; L = 512 10.2 and 7.9, 768 14.5 and 9.4; L = 256 7.6 and 9.8) and four where
    // a thread has four pairs (L = 1000: 24.3 against 20.4, five 27.0 and 31.1 with the
    // copy back)
    if (L < kDeepMinL || L > kDeepMaxL || L % 2 || n < (L > 832 ? 5 : L >= 384 ? 3 : 2)) return false;
    d->tx = d->ty = std::min(16, (L + 15) / 16);
    d->rp = d->full = 0;
    if (meas && L % 64 == 0) {
        // the columns of the tile xy_get_plan reports: 256 x 16 (16 rows: four pairs,
        // 4 rows apart), 128 x 32 (32 rows: four, 8 apart), 64 x 32 (32 rows: two, 16
        // apart).  Cores of whole blocks of rows, one or, from four pairs a thread on, two
        // (ten measured sweeps, one against two: L = 576 3.87 and 3.96 us a sweep, L =
        // 640 7.5 and 5.4, L = 832 7.3 and 5.3), their width again for one region a CU.
        d->rp = L % 256 == 0 ? 4 : L % 128 == 0 ? 8 : 16;
        d->full = L % 128 == 0 ? 4 : 2;
        if (L % 256 != 0) {
            const int P = L / 4;
            d->ty = L > 600 ? L / 64 : L / 32;
            d->tx = L > 600 ? 256 / d->ty : std::min(P / 2, std::max(8192 / L, (P + 11) / 12));
        }
    }
    *nmax = deep_depth(L, d);
    return *nmax > 0;
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
    XY_DEEP(1024, 4);
#undef XY_DEEP
    return hipErrorInvalidValue;
}

template <typename T>
static hipError_t go_deep(const SweepArgs& a, const DeepPlan& d, int n, int me, int phase, double* part, hipStream_t s)
{
    const bool meas = me > 0 && n >= me - phase;    // phase < me
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

// ------------------------------------------------------ four replicas of a quad
// Replica blockIdx.y of a quad: its regions are those of a lattice of its own, read
// from and written to its components of the float4 states (the replicas of a region
// fall on one XCD where a lattice's regions are a multiple of 8, so their stores
// merge in its L2).
template <int NT, int R, int MEAS>
__global__ void __launch_bounds__(NT)
k_deep_quad(const float* __restrict__ src, float* __restrict__ dst, int L, int tx, int ty, int PC, int RY, int hx,
            int hy, uint32_t sweep0, int n, int me, int phase, Params4 p, double* __restrict__ part)
{
    extern __shared__ __align__(16) char smem[];
    const int nb = (int)gridDim.x, b = (int)blockIdx.x, r = (int)blockIdx.y;
    const DeepRegion g = region_of(b, L, tx, ty, PC, RY, hx, hy);
    const Params pr{p.delta[r], p.nbl2e[r]};
    deep_program<float, NT, R, false, false, MEAS, true>(
        src + r, dst + r, g, sweep0, n, me, phase, 0, 0, p.k0[r], p.k1[r], pr, smem,
        [&](int k, double s) { part[((size_t)(4 * k + r) * nb + b) * 8 + threadIdx.x] = s; });
}

// The same with the whole lattice in one workgroup (L = 32): any number of sweeps
// in place; the partial record is the record.
template <int NT, int MEAS>
__global__ void __launch_bounds__(NT)
k_resident_quad(float* __restrict__ st, int L, uint32_t sweep0, int n, int me, Params4 p, xy_obs* __restrict__ obs)
{
    extern __shared__ __align__(16) char smem[];
    const int r = (int)blockIdx.x;
    const Params pr{p.delta[r], p.nbl2e[r]};
    const DeepRegion g{L, L >> 1, L >> 2, 0, 0, L >> 2, L, 0, 0, L >> 2, L};
    deep_program<float, NT, 1, false, true, MEAS, true>(
        st + r, st + r, g, sweep0, n, me, 0, 0, 0, p.k0[r], p.k1[r], pr, smem, [&](int k, double s) {
            // xy_obs: sweep, n_accept, then the six sums, eight bytes each
            const int t = (int)threadIdx.x;
            unsigned long long* o = (unsigned long long*)(obs + (size_t)k * 4 + r);
            if (t < 6) o[2 + t] = (unsigned long long)__double_as_longlong(s);
            else if (t == 6) o[1] = (unsigned long long)s;
            else o[0] = (uint64_t)sweep0 + (uint64_t)(k + 1) * (uint64_t)me;
        });
}

// A quad's replicas share the device, a quarter of it each: 8 x 8 regions.
// Measured, us for ten sweeps, against single sweeps by tiles: L = 96 19.0 (64.8 one
// kernel for the four), L = 256 23.0 (53.9), L = 384 31 (53.2), L = 512 43 (57), L =
// 576 52 (61), L = 640 81 (68).  Beyond L = 384, where a thread has four pairs, two
// sweeps take longer (L = 512 19.3 against 14.1), three less.
constexpr int kDeepQuadMaxL = 576;

bool deep_choose_quad(int L, int64_t n, DeepPlan* d, int* nmax)
{
    if (L < kDeepMinL || L > kDeepQuadMaxL || L % 4 || n < (L > 384 ? 3 : 2)) return false;
    d->rp = d->full = 0;
    d->tx = d->ty = std::min(8, (L + 15) / 16);
    *nmax = deep_depth(L, d);
    return *nmax > 0;
}

template <int NT, int R, int MEAS>
static hipError_t run_deep_quad(const float4* src, float4* dst, int L, uint32_t sweep, const Params4& p,
                                const DeepPlan& d, int n, int me, int phase, double* part, hipStream_t s)
{
    static bool attr_set = false;
    auto kern = k_deep_quad<NT, R, MEAS>;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3(d.tx * d.ty, 4), dim3(NT), deep_lds_bytes(d.PC, d.RY, NT), s, (const float*)src,
                       (float*)dst, L, d.tx, d.ty, d.PC, d.RY, d.hx, d.hy, sweep, n, me, phase, p, part);
    return hipGetLastError();
}

hipError_t launch_deep_quad(const float4* src, float4* dst, int L, uint32_t sweep, const Params4& p, const DeepPlan& d,
                            int n, int me, int phase, double* part, hipStream_t s)
{
    const bool meas = me > 0 && n >= me - phase;    // phase < me
#define XY_DEEP(nt, r)                                                                                           \
    if (deep_fits<nt, r>(d))                                                                                     \
        return meas ? run_deep_quad<nt, r, kMeasQuad>(src, dst, L, sweep, p, d, n, me, phase, part, s)            \
                    : run_deep_quad<nt, r, kMeasNone>(src, dst, L, sweep, p, d, n, me, phase, part, s)
    XY_DEEP(512, 1);
    XY_DEEP(1024, 1);
    XY_DEEP(1024, 2);
    XY_DEEP(1024, 4);
#undef XY_DEEP
    return hipErrorInvalidValue;
}

hipError_t launch_resident_quad(float4* state, int L, uint32_t sweep, const Params4& p, int n, int me, xy_obs* obs,
                                hipStream_t s)
{
    if (L % 4 || (L / 2) * (L / 4) > kDeepPairs<512, 1>) return hipErrorInvalidValue;
    const size_t lds = deep_lds_bytes(L / 4, L, 512);
    if (me > 0 && obs)
        hipLaunchKernelGGL((k_resident_quad<512, kMeasQuad>), dim3(4), dim3(512), lds, s, (float*)state, L, sweep, n, me,
                           p, obs);
    else
        hipLaunchKernelGGL((k_resident_quad<512, kMeasNone>), dim3(4), dim3(512), lds, s, (float*)state, L, sweep, n, 0,
                           p, obs);
    return hipGetLastError();
}

// Workgroup k: record k from its np partial records (fixed order); every `group`
// records share a sweep count, first, first + every, ...
__global__ void __launch_bounds__(256)
k_finalize_many(const double* __restrict__ part, int np, xy_obs* __restrict__ out, uint64_t first, int every, int group)
{
    __shared__ double red[32];
    const int k = (int)blockIdx.x;
    const double s = column_sums(part + (size_t)k * np * 8, np, red);
    put_record(out + k, s, first + (uint64_t)(k / group) * (uint64_t)every, 0ull);
}

hipError_t launch_finalize_many(const double* part, int np, int nrec, xy_obs* out, uint64_t first, int every,
                                hipStream_t s, int group)
{
    hipLaunchKernelGGL(k_finalize_many, dim3(nrec), dim3(256), 0, s, part, np, out, first, every, group);
    return hipGetLastError();
}

}  // namespace xyk
