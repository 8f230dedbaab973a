// xy_runtime.hpp -- runtime helpers shared by the single-lattice and batch front ends.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "xy.h"
#include "xy_launch.hpp"

namespace xyr {

int hip_fail(hipError_t e, const char* what);
// Failure injection (xy_test_inject_failure): true at the launch point that is
// due to fail; the caller then reports hipErrorLaunchFailure without launching.
bool inject_due();
// `expr` (a call returning hipError_t), or an injected launch failure.
#define XY_LAUNCH(expr) (xyr::inject_due() ? hipErrorLaunchFailure : (expr))
bool valid_L(int32_t L);
bool valid_beta_delta(double beta, double delta);
xyk::SweepArgs sweep_args(uint64_t seed, int L, int precision, double beta, double delta);
// The launches of a call of n sweeps on chip with a record every me-th (0: none), `done`
// of them enqueued: the sweeps of the next one and its record interval.  At most about
// a second of work each (2^20 sweeps, 2^30 site updates), so that a long call stays a
// sequence of launches; cut at records, and inside an interval longer than that into
// launches without and a last one with a record of its own last sweep.
struct OnChipLaunch {
    int n, me;
};
inline OnChipLaunch on_chip_launch(int L, int64_t n, int64_t done, int32_t me)
{
    const int64_t w = ((int64_t)1 << 30) / ((int64_t)L * L), most = w < (1 << 20) ? w : (1 << 20);
    const int64_t left = n - done;
    if (me > most) {
        const int64_t until = me - done % me, m = until < left ? until : left;
        return m > most ? OnChipLaunch{(int)most, 0} : OnChipLaunch{(int)m, m == until ? (int)m : 0};
    }
    const int64_t m = me ? most / me * me : most;
    return OnChipLaunch{(int)(m < left ? m : left), me};
}
xy_plan default_plan(int32_t L, int32_t precision);
bool plan_ok(int32_t L, const xy_plan& p);
bool cache_lookup(const char* path, int32_t L, int32_t precision, xy_plan* plan);
const char* env_cache_path();
// xy_attach + xy_sweep on a handle that lives on the stack, with `work` as its
// workspace (zeroed counters first) and the default plan: no host or device
// allocation, no file access.  Arguments as xy_attach / xy_sweep, validated.
int sweep_on_work(uint64_t seed, int32_t L, double beta, double delta, int32_t precision, uint64_t sweep,
                  int64_t n_sweeps, int32_t measure_every, void* state_dev, size_t state_len, void* work,
                  size_t work_len, xy_obs* obs_dev, hipStream_t stream);

}  // namespace xyr
