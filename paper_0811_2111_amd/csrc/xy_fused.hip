// xy_fused.hip -- single-lattice fused sweep: one workgroup per tile, M sweeps per launch.
#include <hip/hip_runtime.h>

#include "xy_launch.hpp"
#include "xy_tile.hpp"
#include "xy_tile1.hpp"

using namespace xyd;

namespace xyk {

// Workgroups are dispatched round-robin over the 8 XCDs (block b -> XCD b % 8).
// Remap so that each XCD works on one contiguous band of tile rows and the halo
// rows two neighbouring tiles share stay in that XCD's L2.
__device__ __forceinline__ int xcd_tile(int b, int ntiles)
{
    if ((ntiles & 7) != 0) return b;
    const int per = ntiles >> 3;
    return (b & 7) * per + (b >> 3);
}

// LDS bytes of a fused launch: the single-sweep tile keeps (cos, sin) only, the
// two-sweep tile also the angles.
template <int TX, int TY, int M, int NT>
constexpr size_t fused_lds()
{
    if constexpr (M == 1) return Tile1<TX, TY, NT>::lds_bytes;
    else return TileShape<TX, TY, M, NT>::lds_bytes;
}

// Lattices whose two buffers (state and ping-pong) together exceed the 256 MiB
// MALL are read back from HBM every sweep; their single-sweep tiles store with
// the non-temporal hint, so the stored rows do not crowd the halo rows the tiles
// beside still have to read out of the L2 (L = 8192 in FP32: 5% less time per
// sweep).  Within the MALL the hint costs more than it saves (L = 4096: 12% more).
constexpr size_t kStreamBytes = (size_t)256 << 20;

// MEAS (single-sweep tiles only): 1 = this sweep is measured, one partial record
// per wave (tile-major); 0 = not measured.  The two-sweep tile takes the mask of
// measured sub-sweeps at run time, one record per tile and sub-sweep.  ST
// (single-sweep tiles only): non-temporal stores.
template <typename T, int TX, int TY, int M, int NT, int MEAS, bool ST>
__global__ void __launch_bounds__(NT)
k_fused(const T* __restrict__ src, T* __restrict__ dst, int L, uint32_t sweep0, uint32_t k0, uint32_t k1, Params p,
        unsigned meas_mask, double* __restrict__ partials)
{
    extern __shared__ __align__(16) char smem[];
    const int tiles_x = L / TX;
    const int ntiles = tiles_x * (L / TY);
    const int b = xcd_tile((int)blockIdx.x, ntiles);
    const int ty = b / tiles_x, tx = b - ty * tiles_x;
    double* red = (double*)(smem + fused_lds<TX, TY, M, NT>());
    if constexpr (M == 1)
        tile1_program<T, TX, TY, NT, MEAS, ST>(src, dst, (unsigned)((size_t)L * L * sizeof(T)), L, tx * TX, ty * TY,
                                           sweep0, k0, k1, p, MEAS != 0, partials + (size_t)b * (NT / 64) * 8, smem,
                                           red);
    else
        tile_program<T, TX, TY, M, NT>(src, dst, L, tx * TX, ty * TY, sweep0, k0, k1, p, meas_mask,
                                       partials + (size_t)b * 8, (size_t)ntiles * 8, smem, red);
}

template <typename T, int TX, int TY, int M, int NT, int MEAS, bool ST>
static hipError_t run_fused_k(const SweepArgs& a, unsigned meas_mask, double* partials, hipStream_t s)
{
    constexpr size_t lds = fused_lds<TX, TY, M, NT>() + (size_t)(NT / 64) * 7 * sizeof(double);
    static bool attr_set = false;
    auto kern = k_fused<T, TX, TY, M, NT, MEAS, ST>;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int ntiles = (a.L / TX) * (a.L / TY);
    const Params p{a.delta, a.nbl2e};
    hipLaunchKernelGGL(kern, dim3(ntiles), dim3(NT), lds, s, (const T*)a.src, (T*)a.dst,
                       a.L, a.sweep, a.key0, a.key1, p, meas_mask, partials);
    return hipGetLastError();
}

template <typename T, int TX, int TY, int M, int NT>
static hipError_t run_fused(const SweepArgs& a, unsigned meas_mask, double* partials, hipStream_t s)
{
    if constexpr (M == 1) {
        const bool st = 2 * (size_t)a.L * (size_t)a.L * sizeof(T) > kStreamBytes;
        if (meas_mask & 1u)
            return st ? run_fused_k<T, TX, TY, M, NT, 1, true>(a, meas_mask, partials, s)
                      : run_fused_k<T, TX, TY, M, NT, 1, false>(a, meas_mask, partials, s);
        return st ? run_fused_k<T, TX, TY, M, NT, 0, true>(a, meas_mask, partials, s)
                  : run_fused_k<T, TX, TY, M, NT, 0, false>(a, meas_mask, partials, s);
    } else {
        return run_fused_k<T, TX, TY, M, NT, -1, false>(a, meas_mask, partials, s);
    }
}

// The tile shapes the autotuner chooses from.
#define XY_FUSED_SHAPES(X) \
    X(64, 16, 1, 256)      \
    X(64, 32, 1, 256)      \
    X(128, 16, 1, 256)     \
    X(128, 32, 1, 256)     \
    X(128, 64, 1, 256)     \
    X(256, 16, 1, 256)     \
    X(256, 32, 1, 256)     \
    X(64, 32, 2, 256)      \
    X(128, 32, 2, 256)

bool fused_supported(int L, int tile_x, int tile_y, int m)
{
    if (L < 4 || (L % 4) != 0 || tile_x <= 0 || tile_y <= 0) return false;
    // buffer descriptors address the FP32 state with 32-bit byte offsets
    if ((long long)L * L * 4 >= (1LL << 32)) return false;
    if (L % tile_x != 0 || L % tile_y != 0) return false;
    if (2 * m > L || m > L / 2) return false;
#define X(tx, ty, mm, nt) \
    if (tile_x == tx && tile_y == ty && m == mm) return true;
    XY_FUSED_SHAPES(X)
#undef X
    return false;
}

int fused_tiles(int L, int tile_x, int tile_y) { return (L / tile_x) * (L / tile_y); }

int fused_records(int L, int tile_x, int tile_y, int m)
{
    // single-sweep tiles: one record per wave of the 256-thread workgroup
    return fused_tiles(L, tile_x, tile_y) * (m == 1 ? 4 : 1);
}

hipError_t launch_fused(const SweepArgs& a, int tile_x, int tile_y, int m, unsigned meas_mask, double* partials,
                        hipStream_t s)
{
#define X(tx, ty, mm, nt)                                                                          \
    if (tile_x == tx && tile_y == ty && m == mm) {                                                 \
        if (a.precision == XY_FP16) return run_fused<__half, tx, ty, mm, nt>(a, meas_mask, partials, s); \
        return run_fused<float, tx, ty, mm, nt>(a, meas_mask, partials, s);               \
    }
    XY_FUSED_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

// ------------------------------------------------------------- ragged tiles
// Single-sweep tiles of 256 x 16 or 128 x 16 sites for any even side.
static int ragged_tiles(int L, int tile_x) { return ((L + tile_x - 1) / tile_x) * ((L + 15) / 16); }

int ragged_records(int L, int tile_x) { return 4 * ragged_tiles(L, tile_x); }

int ragged_tile_x(int L)
{
    if (L < 256 || L % 2 || (long long)L * L * 4 >= (1LL << 32)) return 0;
    // Sites the tiles cover, times what each shape costs: at L = 4096 the 128 x 16
    // tiles take 8% longer (33.2 against 30.7 us a sweep: half as much work for each
    // tile's loads and barriers), at L = 1024 7% less (4.97 against 5.35: the 256 x 16
    // tiles are one workgroup a CU, with nothing to run while it waits).
    const double w = L <= 1408 ? 0.93 : 1.08;
    return ragged_tiles(L, 128) * 0.5 * w < ragged_tiles(L, 256) ? 128 : 256;
}

// ODD: L % 4 == 2.  Tiles inside the lattice take the program without bounds, which
// interleaves a thread's Philox chains.  Unmeasured, the last tiles are moved back
// inside instead of cut off (both tiles then write the overlap, the same values),
// down the lattice and, where pairs stay aligned, along it.
template <typename T, int TX, int MEAS, bool ST, bool ODD>
__global__ void __launch_bounds__(256)
k_ragged(const T* __restrict__ src, T* __restrict__ dst, int L, uint32_t sweep, uint32_t k0, uint32_t k1, Params p,
         double* __restrict__ partials)
{
    extern __shared__ __align__(16) char smem[];
    const int tiles_x = (L + TX - 1) / TX, ntiles = tiles_x * ((L + 15) / 16);
    const int b = xcd_tile((int)blockIdx.x, (int)gridDim.x);    // a grid of a multiple of 8
    if (b >= ntiles) return;
    const int ty = b / tiles_x;
    int x0 = (b - ty * tiles_x) * TX, y0 = ty * 16;
    if constexpr (MEAS == 0) {
        y0 = min(y0, L - 16);
        if constexpr (!ODD) x0 = min(x0, L - TX);
    }
    const unsigned bytes = (unsigned)((size_t)L * L * sizeof(T));
    double* part = partials + (size_t)b * 4 * 8;
    constexpr int odd = ODD ? kOdd : 0;
    if (x0 + TX <= L && y0 + 16 <= L)
        tile1_program<T, TX, 16, 256, MEAS, ST, odd>(src, dst, bytes, L, x0, y0, sweep, k0, k1, p, MEAS != 0, part,
                                                     smem, nullptr);
    else if constexpr (MEAS != 0 || ODD)
        tile1_program<T, TX, 16, 256, MEAS, ST, odd | kPart>(src, dst, bytes, L, x0, y0, sweep, k0, k1, p, MEAS != 0,
                                                             part, smem, nullptr);
}

template <typename T, int TX, int MEAS, bool ST, bool ODD>
static hipError_t run_ragged_k(const SweepArgs& a, double* part, hipStream_t s)
{
    constexpr size_t lds = Tile1<TX, 16, 256>::lds_bytes;
    static bool attr_set = false;
    auto kern = k_ragged<T, TX, MEAS, ST, ODD>;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const Params p{a.delta, a.nbl2e};
    hipLaunchKernelGGL(kern, dim3((unsigned)((ragged_tiles(a.L, TX) + 7) & ~7)), dim3(256), lds, s, (const T*)a.src,
                       (T*)a.dst, a.L, a.sweep, a.key0, a.key1, p, part);
    return hipGetLastError();
}

template <typename T, int TX, bool ST, bool ODD>
static hipError_t run_ragged(const SweepArgs& a, bool meas, double* part, hipStream_t s)
{
    return meas ? run_ragged_k<T, TX, 2, ST, ODD>(a, part, s) : run_ragged_k<T, TX, 0, ST, ODD>(a, part, s);
}

template <typename T, bool ODD>
static hipError_t pick_ragged(const SweepArgs& a, int tile_x, bool meas, double* part, hipStream_t s)
{
    if (tile_x == 128) return run_ragged<T, 128, false, ODD>(a, meas, part, s);
    const bool st = 2 * (size_t)a.L * (size_t)a.L * sizeof(T) > kStreamBytes;
    return st ? run_ragged<T, 256, true, ODD>(a, meas, part, s) : run_ragged<T, 256, false, ODD>(a, meas, part, s);
}

hipError_t launch_ragged(const SweepArgs& a, int tile_x, bool meas, double* part, hipStream_t s)
{
    if (ragged_tile_x(a.L) == 0 || (tile_x != 128 && tile_x != 256)) return hipErrorInvalidValue;
    if (a.L % tile_x == 0 && !meas)    // whole tiles
        return launch_fused(a, tile_x, 16, 1, 0u, part, s);
    if (a.precision == XY_FP16)
        return a.L % 4 ? pick_ragged<__half, true>(a, tile_x, meas, part, s)
                       : pick_ragged<__half, false>(a, tile_x, meas, part, s);
    return a.L % 4 ? pick_ragged<float, true>(a, tile_x, meas, part, s)
                   : pick_ragged<float, false>(a, tile_x, meas, part, s);
}

}  // namespace xyk
