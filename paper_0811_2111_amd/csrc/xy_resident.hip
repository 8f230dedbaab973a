// xy_resident.hip -- single-lattice sweeps with the whole lattice on chip
// (L <= 128): every sweep of a call in one launch of one workgroup.
#include <hip/hip_runtime.h>

#include "xy_launch.hpp"
#include "xy_resident.hpp"

using namespace xyd;

namespace xyk {

template <typename T, int NT, int R, bool ODD, int MEAS>
__global__ void __launch_bounds__(NT)
k_resident(const T* __restrict__ src, T* __restrict__ dst, int L, uint32_t sweep0, int n, int me, uint32_t k0,
           uint32_t k1, Params p, xy_obs* __restrict__ obs)
{
    extern __shared__ __align__(16) char smem[];
    resident_program<T, NT, R, ODD, MEAS>(src, dst, L, sweep0, n, me, k0, k1, p, obs, smem);
}

bool resident_supported(int L) { return L >= 4 && L <= kResidentMaxL && L % 4 == 0; }

template <typename T, int NT, int R, bool ODD, int MEAS>
static hipError_t run_resident(const SweepArgs& a, int n, int me, xy_obs* obs, hipStream_t s)
{
    static bool attr_set = false;
    auto kern = k_resident<T, NT, R, ODD, MEAS>;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const Params p{a.delta, a.nbl2e};
    hipLaunchKernelGGL(kern, dim3(1), dim3(NT), resident_lds_bytes(a.L, NT), s, (const T*)a.src, (T*)a.dst, a.L,
                       a.sweep, n, me, a.key0, a.key1, p, obs);
    return hipGetLastError();
}

// The smallest workgroup that holds the lattice with one pair a thread, and more
// pairs a thread beyond 1024 threads.
#define XY_RES(nt, r) \
    if (resident_fits<nt, r>(a.L)) return run_resident<T, nt, r, ODD, MEAS>(a, n, me, obs, s)
template <typename T, bool ODD, int MEAS>
static hipError_t pick_resident(const SweepArgs& a, int n, int me, xy_obs* obs, hipStream_t s)
{
    XY_RES(256, 1);
    XY_RES(512, 1);
    XY_RES(1024, 1);
    XY_RES(1024, 2);
    if constexpr (MEAS == kMeasOwn) {
        XY_RES(1024, 4);
        XY_RES(1024, 8);
    }
    return hipErrorInvalidValue;
}
#undef XY_RES

hipError_t launch_resident(const SweepArgs& a, int n, int me, xy_obs* obs, hipStream_t s)
{
    if (!resident_supported(a.L) || n < 0) return hipErrorInvalidValue;
    if (a.precision == XY_FP16) return pick_resident<__half, false, kMeasOwn>(a, n, me, obs, s);
    return pick_resident<float, false, kMeasOwn>(a, n, me, obs, s);
}

hipError_t launch_resident_any(const SweepArgs& a, int n, int me, xy_obs* obs, hipStream_t s)
{
    if (a.L < 4 || a.L % 2 || n < 0) return hipErrorInvalidValue;
    if (a.precision == XY_FP16)
        return a.L % 4 ? pick_resident<__half, true, kMeasPair>(a, n, me, obs, s)
                       : pick_resident<__half, false, kMeasPair>(a, n, me, obs, s);
    return a.L % 4 ? pick_resident<float, true, kMeasPair>(a, n, me, obs, s)
                   : pick_resident<float, false, kMeasPair>(a, n, me, obs, s);
}

}  // namespace xyk
