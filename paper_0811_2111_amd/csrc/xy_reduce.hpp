// xy_reduce.hpp -- the workgroup-level step of the fixed-order FP64 reductions,
// shared by the sweep's record reduction and the hybrid Monte Carlo sums.
#pragma once

#include "xy.h"
#include "xy_device.hpp"

namespace xyd {

// Sums of n >= 1 records (8 doubles each, back to back in global memory or LDS) by a
// workgroup of NT threads: thread t adds column t % 8 of the records t / 8, t / 8 +
// NT / 8, ..., so that a wave reads 512 bytes in a row; then the lanes of a wave with
// one column are added, then the waves in order.  Threads 0 .. 7 get the total of
// their column.  `red`: NT / 8 doubles of LDS, free again after the caller's next
// barrier.  These kernels are one chain of latencies, hence the loads of eight
// records in flight (past the end: the last one again, dropped) and one value a
// thread to exchange: 32768 records (two levels) 8.4 us, 9.9 with seven values a
// thread; 16384 5.2 and 6.1; 2016 by one workgroup of 1024 threads 2.6, of 256 with
// seven values each 3.1.
template <int NT = 256>
__device__ __forceinline__ double column_sums(const double* rec, int n, double* red)
{
    const int t = (int)threadIdx.x, c = t & 7;
    double s = 0.0;
    for (int i = t >> 3; i < n; i += NT) {
        double v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = rec[(size_t)min(i + k * (NT / 8), n - 1) * 8 + c];
#pragma unroll
        for (int k = 0; k < 8; ++k) s += i + k * (NT / 8) < n ? v[k] : 0.0;
    }
    s += dpp_f64<0x128>(s);   // row_ror:8
    s = swap16_sum(s, s);
    s = swap32_sum(s, s);
    if ((t & 63) < 8) red[(t >> 6) * 8 + c] = s;
    __syncthreads();
    s = 0.0;
    if (t < 8)
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) s += red[w * 8 + t];
    return s;
}

// Threads 0 .. 7 with their column's total: the observable record.
__device__ __forceinline__ void put_record(xy_obs* __restrict__ out, double s, uint64_t sweep_after,
                                           unsigned long long more_accepts)
{
    // xy_obs: sweep, n_accept, then the six sums, eight bytes each
    const int t = (int)threadIdx.x;
    unsigned long long* o = (unsigned long long*)out;
    if (t < 6) o[2 + t] = (unsigned long long)__double_as_longlong(s);
    else if (t == 6) o[1] = more_accepts + (unsigned long long)s;
    else if (t == 7) o[0] = sweep_after;
}

}  // namespace xyd
