// xy_resident.hpp -- a whole small lattice in one workgroup for every sweep of a
// call: the WRAP form of xy_deep.hpp, with no halo and no HBM traffic between
// sweeps.  A measured sweep's record is written by the workgroup itself.
#pragma once

#include "xy_deep.hpp"

namespace xyd {

constexpr int kResidentMaxL = 128;

// Whether NT threads with R pairs each hold the lattice's pairs of one colour and row parity.
template <int NT, int R>
__host__ __device__ constexpr bool resident_fits(int L) { return (L / 2) * ((L / 2 + 1) / 2) <= kDeepPairs<NT, R>; }

__host__ __device__ constexpr size_t resident_lds_bytes(int L, int nt)
{
    return deep_lds_bytes((L / 2 + 1) / 2, L, nt);
}

// n sweeps of the L x L lattice in src (state layout) starting at sweep index
// sweep0, result in dst (may equal src).  me > 0 and obs != NULL: after the j-th
// sweep of the call (j = 1 .. n) with j % me == 0 the record j / me - 1 goes to
// obs, its terms gathered as MEAS says (kMeasOwn or kMeasPair).  resident_fits<NT, R>(L); smem: resident_lds_bytes(L, NT).
template <typename T, int NT, int R, bool ODD, int MEAS>
__device__ __forceinline__ void resident_program(const T* __restrict__ src, T* __restrict__ dst, int L,
                                                 uint32_t sweep0, int n, int me, uint32_t k0, uint32_t k1,
                                                 const Params& p, xy_obs* __restrict__ obs, char* smem)
{
    DeepRegion g;
    g.L = L;
    g.Hh = L >> 1;
    g.P = (g.Hh + 1) >> 1;
    g.ps = g.ys = g.hx = g.hy = 0;
    g.PC = g.cp = g.P;
    g.RY = g.cr = L;
    if (obs == nullptr) me = 0;
    deep_program<T, NT, R, ODD, true, MEAS, false>(src, dst, g, sweep0, n, me, 0, 0, 0, k0, k1, p, smem, [&](int k, double s) {
        // xy_obs: sweep, n_accept, then the six sums, eight bytes each
        const int t = (int)threadIdx.x;
        const uint64_t after = (uint64_t)sweep0 + (uint64_t)(k + 1) * (uint64_t)me;
        unsigned long long* o = (unsigned long long*)(obs + k);
        if (t < 6) o[2 + t] = (unsigned long long)__double_as_longlong(s);
        else if (t == 6) o[1] = (unsigned long long)s;
        else o[0] = after;
    });
}

}  // namespace xyd
