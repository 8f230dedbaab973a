// xy_quad.hip -- four replicas of one lattice in one float4 state: hot start,
// fused sweeps, sweeps of the four lattices apart, measurement records, and the
// xy_quad_* C ABI.  (Several sweeps per launch: xy_deep.hip.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <new>

#include "xy.h"
#include "xy_launch.hpp"
#include "xy_runtime.hpp"
#include "xy_tile4.hpp"

using namespace xyd;

namespace xyk {

namespace {

// Hot start: replica r of entry (c, y, k) takes u of word X0 (even k) or X2 (odd
// k) of Philox(0, c, 1, y P + k/2) keyed by seed_r, exactly as a single lattice
// with seed_r; cold start: 0.
__global__ void __launch_bounds__(256) k_quad_init(float4* __restrict__ st, int L, Params4 p, int hot)
{
    const int Hh = L >> 1, P = (Hh + 1) >> 1;
    const int j = blockIdx.x * 64 + threadIdx.x;
    const int y = blockIdx.y * 4 + threadIdx.y;
    const int c = blockIdx.z;
    if (j >= P || y >= L) return;
    float4* row = st + ((size_t)c * L + y) * Hh;
    const int ka = 2 * j, kb = 2 * j + 1;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
    if (hot) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const u32x4 w = philox10(0u, (uint32_t)c, 1u, (uint32_t)(y * P + j), p.k0[r], p.k1[r]);
            f4set(a, r, u01(w.x));
            f4set(b, r, u01(w.z));
        }
    }
    row[ka] = a;
    if (kb < Hh) row[kb] = b;
}

__global__ void __launch_bounds__(256) k_quad_copy(const float4* __restrict__ src, float4* __restrict__ dst, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) dst[i] = src[i];
}

__device__ __forceinline__ int xcd_tile4(int b, int ntiles)
{
    if ((ntiles & 7) != 0) return b;
    const int per = ntiles >> 3;
    return (b & 7) * per + (b >> 3);
}

template <int TX, int TY, bool MEAS, bool IN, bool OUT>
__global__ void __launch_bounds__(256)
k_quad_fused(const void* __restrict__ src, void* __restrict__ dst, int L, uint32_t sweep, Params4 p,
             double* __restrict__ partials)
{
    extern __shared__ __align__(16) char smem[];
    const int tiles_x = L / TX;
    const int ntiles = tiles_x * (L / TY);
    const int b = xcd_tile4((int)blockIdx.x, ntiles);
    const int ty = b / tiles_x, tx = b - ty * tiles_x;
    tile4_program<TX, TY, 256, MEAS, IN, OUT>(src, dst, (unsigned)((size_t)L * L * sizeof(float4)), L, tx * TX, ty * TY, sweep,
                                     p, partials + (size_t)b * 4 * 8, (size_t)ntiles * 4, smem);
}

template <int TX, int TY, bool MEAS, bool IN = false, bool OUT = false>
hipError_t run_quad(const void* src, void* dst, int L, uint32_t sweep, const Params4& p, double* partials,
                    hipStream_t s)
{
    constexpr size_t lds = Tile4<TX, TY, 256>::lds_bytes;
    static bool attr_set = false;
    auto kern = k_quad_fused<TX, TY, MEAS, IN, OUT>;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int ntiles = (L / TX) * (L / TY);
    hipLaunchKernelGGL(kern, dim3(ntiles), dim3(256), lds, s, src, dst, L, sweep, p, partials);
    return hipGetLastError();
}

// One sweep of the four lattices of a quad back to back (blockIdx.y: the replica)
// by TX x 16 tiles; the last ones are cut off at the lattice's edge when measured
// and moved back inside otherwise.  Records as tile4_program's: each pair's terms by
// themselves, a record per wave.
//
// Bound by the vector unit, as the single-lattice tiles.  A float4 tile moves 16
// bytes of (cos, sin) through LDS for every 4 updates' one, holds two to three times the
// registers and runs three workgroups a CU to this one's four: measured, us a sweep
// of all four, k_quad_fused against this: L = 1024 13.5 and 12.0, L = 2048 42.5 and
// 32, L = 4096 160 and 123.5 (from L = 2800 the strips of xy_walk.hip, 115); measured sweeps 18 and 16 at L = 1024, 230 and 140 at
// L = 4096.
template <int TX, bool MEAS, bool ST>
__global__ void __launch_bounds__(256)
k_planes(const float* __restrict__ src, float* __restrict__ dst, int L, uint32_t sweep, Params4 p,
         double* __restrict__ partials)
{
    extern __shared__ __align__(16) char smem[];
    const int tiles_x = (L + TX - 1) / TX, ntiles = tiles_x * ((L + 15) / 16);
    const int b = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);   // a multiple of 8
    if (b >= ntiles) return;
    const int r = (int)blockIdx.y;
    const int ty = b / tiles_x;
    int x0 = (b - ty * tiles_x) * TX, y0 = ty * 16;
    if constexpr (!MEAS) {
        y0 = min(y0, L - 16);
        x0 = min(x0, L - TX);
    }
    const size_t n = (size_t)L * L;
    const Params pr{p.delta[r], p.nbl2e[r]};
    double* part = partials + ((size_t)r * ntiles + b) * 4 * 8;
    if (!MEAS || (x0 + TX <= L && y0 + 16 <= L))
        tile1_program<float, TX, 16, 256, MEAS ? 3 : 0, ST>(src + r * n, dst + r * n, (unsigned)(n * 4), L, x0, y0,
                                                            sweep, p.k0[r], p.k1[r], pr, MEAS, part, smem, nullptr);
    else if constexpr (MEAS)
        tile1_program<float, TX, 16, 256, 3, ST, kPart>(src + r * n, dst + r * n, (unsigned)(n * 4), L, x0, y0, sweep,
                                                        p.k0[r], p.k1[r], pr, true, part, smem, nullptr);
}

template <int TX, bool MEAS, bool ST>
hipError_t run_planes(const float* src, float* dst, int L, uint32_t sweep, const Params4& p, double* part,
                      hipStream_t s)
{
    constexpr size_t lds = Tile1<TX, 16, 256>::lds_bytes;
    static bool attr_set = false;
    auto kern = k_planes<TX, MEAS, ST>;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const unsigned tiles = (unsigned)(((L + TX - 1) / TX) * ((L + 15) / 16));
    hipLaunchKernelGGL(kern, dim3((tiles + 7) & ~7u, 4), dim3(256), lds, s, src, dst, L, sweep, p, part);
    return hipGetLastError();
}

// Sites the tiles cover, the 128 x 16 ones at 8% more each (as for a single lattice).
int planes_tile_x(int L)
{
    const int t128 = (L + 127) / 128, t256 = (L + 255) / 256;
    return t128 * 0.54 < t256 ? 128 : 256;
}
int planes_records(int L) { return 4 * ((L + planes_tile_x(L) - 1) / planes_tile_x(L)) * ((L + 15) / 16); }

hipError_t launch_planes(const float* src, float* dst, int L, uint32_t sweep, const Params4& p, bool meas,
                         double* part, hipStream_t s)
{
    if (!meas && walk_quad_supported(L)) return launch_walk_quad(src, dst, L, sweep, p, s);
    const bool st = 2 * (size_t)L * L * sizeof(float4) > (size_t)256 << 20;     // beyond the MALL
#define X(tx)                                                                                               \
    if (planes_tile_x(L) == tx)                                                                             \
        return meas ? st ? run_planes<tx, true, true>(src, dst, L, sweep, p, part, s)               \
                         : run_planes<tx, true, false>(src, dst, L, sweep, p, part, s)              \
                    : st ? run_planes<tx, false, true>(src, dst, L, sweep, p, part, s)              \
                         : run_planes<tx, false, false>(src, dst, L, sweep, p, part, s)
    X(128);
    X(256);
#undef X
    return hipErrorInvalidValue;
}

}  // namespace

// Tile shapes (256 threads, TX/4 pairs per row; one or two pair items per thread
// and half-sweep, each item eight independent updates).
#define XY_QUAD_SHAPES(X) \
    X(32, 16)             \
    X(64, 8)              \
    X(64, 16)             \
    X(128, 4)             \
    X(128, 8)

static bool quad_shape_ok(int L, int tx, int ty)
{
#define X(a, b) \
    if (tx == a && ty == b) return L % a == 0 && L % b == 0;
    XY_QUAD_SHAPES(X)
#undef X
    return false;
}

// One sweep between the float4 layout and the four lattices (`in`: src holds the
// lattices, else dst does), by the default tiles.
static hipError_t launch_quad_convert(const void* src, void* dst, int L, uint32_t sweep, const Params4& p, bool in,
                                      bool meas, double* part, hipStream_t s)
{
#define X(a, b)                                                                                   \
    return in ? meas ? run_quad<a, b, true, true, false>(src, dst, L, sweep, p, part, s)          \
                     : run_quad<a, b, false, true, false>(src, dst, L, sweep, p, part, s)         \
              : meas ? run_quad<a, b, true, false, true>(src, dst, L, sweep, p, part, s)          \
                     : run_quad<a, b, false, false, true>(src, dst, L, sweep, p, part, s)
    if (L % 128 == 0) X(128, 8);
    X(32, 16);
#undef X
}

static hipError_t launch_quad(const float4* src, float4* dst, int L, int tx, int ty, uint32_t sweep,
                              const Params4& p, bool meas, double* partials, hipStream_t s)
{
#define X(a, b)                                                                                   \
    if (tx == a && ty == b)                                                                       \
        return meas ? run_quad<a, b, true>(src, dst, L, sweep, p, partials, s)                    \
                    : run_quad<a, b, false>(src, dst, L, sweep, p, partials, s);
    XY_QUAD_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace xyk

// ----------------------------------------------------------------------- C ABI

namespace {

constexpr uint32_t kQuadMagic = 0x51554144u;   // "QUAD"
constexpr int kQuadHmcSteps = 4;               // largest steps-per-pass setting

size_t quad_state_bytes(int L) { return (size_t)L * (size_t)L * sizeof(float4); }
// one partial record per wave (4 per 256-thread tile) and replica; the smallest
// tiles (32 x 16, 64 x 8, 128 x 4) hold 512 sites
size_t quad_max_records(int L) { return (size_t)L * (size_t)L / 512 * 4 * 4; }
size_t quad_chunks(int L) { return (quad_max_records(L) / 4 + 255) / 256 * 4; }
// ping-pong state, 256 bytes for the finalize's arrival counter, partials, chunks
size_t quad_work_bytes(int L)
{
    return ((quad_state_bytes(L) + 255) & ~(size_t)255) + 256 +
           (quad_max_records(L) + quad_chunks(L)) * 8 * sizeof(double);
}

bool quad_L_ok(int32_t L)
{
    // float4 entries addressed with 32-bit byte offsets; tiles need L % 32 == 0
    return L >= 32 && L % 32 == 0 && (long long)L * L * 16 < (1LL << 32);
}

}  // namespace

struct xy_quad {
    uint32_t magic;
    int32_t L;
    uint64_t seed[4];
    double beta[4], delta[4];
    float4* state;
    float4* pingpong;
    double* partials;
    double* chunks;
    unsigned* arrive;      // arrival counter of the one-launch record reduction (zero between calls)
    hipStream_t stream;
    uint64_t sweep;
    int32_t tile_x, tile_y;
    bool tile_set;         // the caller chose the tile: every sweep takes it
    int32_t hmc_steps;     // leap-frog steps per pass of xy_quad_hmc (1 .. 4; 0: the library's choice)
};

static bool quad_live(const xy_quad* q) { return q && q->magic == kQuadMagic; }

static xyd::Params4 quad_params(const xy_quad* q)
{
    xyd::Params4 p;
    for (int r = 0; r < 4; ++r) {
        const xyk::SweepArgs a = xyr::sweep_args(q->seed[r], q->L, XY_FP32, q->beta[r], q->delta[r]);
        p.delta[r] = a.delta;
        p.nbl2e[r] = a.nbl2e;
        p.k0[r] = a.key0;
        p.k1[r] = a.key1;
    }
    return p;
}

// A launch that the state needs to agree with the counter, also after a failed one:
// launched again if it fails.
template <typename F>
static void quad_finish(int& rc, const char* what, F launch)
{
    hipError_t e = rc == XY_OK ? XY_LAUNCH(launch()) : launch();
    if (e == hipSuccess) return;
    if (rc == XY_OK) rc = xyr::hip_fail(e, what);
    (void)launch();
}

// Every sweep in one launch of four workgroups (L = 32; long calls in several).
static int quad_resident_sweeps(xy_quad* q, int64_t n_sweeps, int32_t me, xy_obs* obs)
{
    const xyd::Params4 p = quad_params(q);
    for (int64_t done = 0; done < n_sweeps;) {
        const xyr::OnChipLaunch c = xyr::on_chip_launch(q->L, n_sweeps, done, me);
        hipError_t e = XY_LAUNCH(xyk::launch_resident_quad(q->state, q->L, (uint32_t)q->sweep, p, c.n, c.me,
                                                           c.me ? obs + done / me * 4 : nullptr, q->stream));
        if (e != hipSuccess) return xyr::hip_fail(e, "xy_quad_sweep: launch");
        q->sweep += (uint64_t)c.n;
        done += c.n;
    }
    return XY_OK;
}

// Passes of several sweeps from `state` to the ping-pong buffer and back, an even
// number of them, as a single lattice's (deep_sweeps of the lattice calls).
static int quad_deep_sweeps(xy_quad* q, const xyk::DeepPlan& plan, int nmax, int64_t n_sweeps, int32_t me, xy_obs* obs)
{
    const xyd::Params4 p = quad_params(q);
    const int np = plan.tx * plan.ty, room = (int)(quad_max_records(q->L) / 4 / np);
    // a pass measures no more sweeps than the workspace holds records of
    if (me && (int64_t)room * me < nmax) nmax = room * me;
    const int64_t passes = ((n_sweeps + nmax - 1) / nmax + 1) / 2 * 2;
    const uint64_t base = q->sweep;
    int held = 0;            // sweeps whose partials wait in the workspace
    int64_t out = 0, j = 0;  // sweeps whose records are written, sweeps done
    auto flush = [&] {
        if (held == 0) return hipSuccess;
        hipError_t e = xyk::launch_finalize_many(q->partials, np, 4 * held, obs + out * 4,
                                                 base + (uint64_t)(out + 1) * (uint64_t)me, me, q->stream, 4);
        if (e == hipSuccess) {
            out += held;
            held = 0;
        }
        return e;
    };
    for (int64_t k = 0; k < passes; ++k) {
        const int n = (int)(n_sweeps / passes + (k < n_sweeps % passes));
        const int phase = me ? (int)(j % me) : 0, nrec = me ? (int)((j + n) / me - j / me) : 0;
        hipError_t e = held > 0 && held + nrec > room ? XY_LAUNCH(flush()) : hipSuccess;
        if (e == hipSuccess) {
            xyk::DeepPlan d = plan;
            e = xyk::deep_region(q->L, n, &d)
                    ? XY_LAUNCH(xyk::launch_deep_quad((k & 1) ? q->pingpong : q->state,
                                                      (k & 1) ? q->state : q->pingpong, q->L, (uint32_t)q->sweep, p, d,
                                                      n, me, phase, q->partials + (size_t)held * 4 * np * 8, q->stream))
                    : hipErrorInvalidValue;
        }
        if (e != hipSuccess) {
            const int rc = xyr::hip_fail(e, "xy_quad_sweep: launch");
            (void)flush();
            if (k & 1)       // so that the state agrees with the counter
                (void)hipMemcpyAsync(q->state, q->pingpong, quad_state_bytes(q->L), hipMemcpyDeviceToDevice, q->stream);
            return rc;
        }
        held += nrec;
        j += n;
        q->sweep += (uint64_t)n;
    }
    hipError_t e = held > 0 ? XY_LAUNCH(flush()) : hipSuccess;
    if (e == hipSuccess) return XY_OK;
    const int rc = xyr::hip_fail(e, "xy_quad_sweep: finalize");
    (void)flush();
    return rc;
}

// Single sweeps of the four lattices apart.  The first sweep writes them (into the
// second buffer), the last reads them; a copy takes the place of the last where
// n_sweeps is odd, of both where every sweep is measured.  The sweeps between are an
// even number, so the angles end in the caller's buffer.
static int quad_plane_sweeps(xy_quad* q, int64_t n_sweeps, int32_t me, xy_obs* obs)
{
    const xyd::Params4 p = quad_params(q);
    auto measured = [&](int64_t j) { return me > 0 && j % me == 0; };     // j = 1-based sweep in call
    const bool first = (n_sweeps & 1) || !measured(1), last = !(n_sweeps & 1) && first;
    int where = 0;           // the angles: 0 state, 1 lattices in pingpong, 2 lattices in state
    int64_t j = 0;
    auto sweep = [&](hipError_t e, int to, int nrec) {
        if (e != hipSuccess) return e;
        where = to;
        ++j;
        q->sweep += 1;
        if (!measured(j)) return hipSuccess;
        return XY_LAUNCH(xyk::launch_finalize_quad(q->partials, nrec, obs + (j / me - 1) * 4, q->sweep, q->chunks,
                                                   q->arrive, q->stream));
    };
    auto convert = [&](bool in) {
        const int tiles = (q->L / q->tile_x) * (q->L / q->tile_y);
        return sweep(XY_LAUNCH(xyk::launch_quad_convert(in ? q->pingpong : q->state, in ? q->state : q->pingpong, q->L,
                                                        (uint32_t)q->sweep, p, in, measured(j + 1), q->partials,
                                                        q->stream)),
                     in ? 0 : 1, 4 * tiles);
    };
    hipError_t e;
    if (first) {
        e = convert(false);
    } else {
        e = XY_LAUNCH(xyk::launch_quad_split(q->state, (float*)q->pingpong, q->L, q->stream));
        if (e == hipSuccess) where = 1;
    }
    while (e == hipSuccess && j < n_sweeps - (last ? 1 : 0)) {
        const bool back = where == 1;
        e = sweep(XY_LAUNCH(xyk::launch_planes((const float*)(back ? q->pingpong : q->state),
                                               (float*)(back ? q->state : q->pingpong), q->L, (uint32_t)q->sweep, p,
                                               measured(j + 1), q->partials, q->stream)),
                  back ? 2 : 1, xyk::planes_records(q->L));
    }
    if (e == hipSuccess && last) e = convert(true);
    int rc = e == hipSuccess ? XY_OK : xyr::hip_fail(e, "xy_quad_sweep: launch");
    // also after a failed launch, so that the state agrees with the counter
    if (where == 2)
        (void)hipMemcpyAsync(q->pingpong, q->state, quad_state_bytes(q->L), hipMemcpyDeviceToDevice, q->stream);
    if (where != 0)
        quad_finish(rc, "xy_quad_sweep: launch",
                    [&] { return xyk::launch_quad_join((const float*)q->pingpong, q->state, q->L, q->stream); });
    return rc;
}

extern "C" {

int xy_quad_state_bytes(int32_t L, size_t* state, size_t* workspace)
{
    if (!quad_L_ok(L)) return XY_EINVAL;
    if (state) *state = quad_state_bytes(L);
    if (workspace) *workspace = quad_work_bytes(L);
    return XY_OK;
}

int xy_quad_init(xy_quad** out, const uint64_t* seeds, int32_t L, const double* beta, const double* delta,
                 int32_t start, void* state_dev, size_t state_len, void* work_dev, size_t work_len, void* hip_stream)
{
    if (!out) return XY_ESTATE;
    *out = nullptr;
    if (!seeds || !beta || !delta || !state_dev || !work_dev) return XY_ESTATE;
    if (!quad_L_ok(L) || (start != XY_HOT && start != XY_COLD)) return XY_EINVAL;
    for (int r = 0; r < 4; ++r)
        if (!xyr::valid_beta_delta(beta[r], delta[r])) return XY_EINVAL;
    if (state_len < quad_state_bytes(L) || work_len < quad_work_bytes(L)) return XY_ESIZE;
    xy_quad* q = new (std::nothrow) xy_quad();
    if (!q) return XY_ENOMEM;
    q->magic = kQuadMagic;
    q->L = L;
    for (int r = 0; r < 4; ++r) {
        q->seed[r] = seeds[r];
        q->beta[r] = beta[r];
        q->delta[r] = delta[r];
    }
    q->state = (float4*)state_dev;
    char* w = (char*)work_dev;
    q->pingpong = (float4*)w;
    w += (quad_state_bytes(L) + 255) & ~(size_t)255;
    q->arrive = (unsigned*)w;
    w += 256;
    q->partials = (double*)w;
    q->chunks = q->partials + quad_max_records(L) * 8;
    q->stream = (hipStream_t)hip_stream;
    q->sweep = 0;
    q->tile_x = L % 128 == 0 ? 128 : 32;
    q->tile_y = L % 128 == 0 ? 8 : 16;
    q->tile_set = false;
    q->hmc_steps = 0;
    const int Hh = L / 2, P = (Hh + 1) / 2;
    hipLaunchKernelGGL(xyk::k_quad_init, dim3((P + 63) / 64, (L + 3) / 4, 2), dim3(64, 4), 0, q->stream, q->state, L,
                       quad_params(q), start == XY_HOT ? 1 : 0);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = xyk::launch_zero_u64((unsigned long long*)q->arrive, 4, q->stream);
    if (e != hipSuccess) {
        q->magic = 0;
        delete q;
        return xyr::hip_fail(e, "xy_quad_init: launch");
    }
    *out = q;
    return XY_OK;
}

int xy_quad_sweep(xy_quad* q, int64_t n_sweeps, int32_t measure_every, xy_obs* obs_dev)
{
    if (!quad_live(q)) return XY_ESTATE;
    if (n_sweeps < 0 || measure_every < 0) return XY_EINVAL;
    if (q->sweep + (uint64_t)n_sweeps >= 0xffffffffull) return XY_ERANGE;
    const bool meas = measure_every > 0 && obs_dev != nullptr && measure_every <= n_sweeps;
    // Where no tile was asked for: the whole quad in four workgroups, passes of
    // several sweeps, or single sweeps of the lattices apart.  A single sweep gains
    // nothing from the latter two, nor do two unmeasured ones from L = 384 on (13.3 us
    // against 14.2; L = 608 21.5 and 24.7, 4096 330 and 343; L = 320 13.2 and 12.8) and
    // four up to L = 1024 (58.0 and 61.4; L = 1536 109 and 92) where the first and last
    // sweep's tiles are the ones of one kernel: they need no copy back.
    const bool short_even = !meas && ((n_sweeps == 2 && q->L >= 384) ||
                                      (n_sweeps == 4 && q->L % 128 == 0 && q->L >= 640 && q->L <= 1024));
    if (!q->tile_set && n_sweeps > 0 && !short_even) {
        const int32_t me = meas ? measure_every : 0;
        xyk::DeepPlan plan;
        int nmax;
        if (q->L == 32) return quad_resident_sweeps(q, n_sweeps, me, obs_dev);
        if (xyk::deep_choose_quad(q->L, n_sweeps, &plan, &nmax))
            return quad_deep_sweeps(q, plan, nmax, n_sweeps, me, obs_dev);
        if (n_sweeps > 1 && q->L >= 256) return quad_plane_sweeps(q, n_sweeps, me, obs_dev);
    }
    const xyd::Params4 p = quad_params(q);
    const int ntiles = (q->L / q->tile_x) * (q->L / q->tile_y);
    const int nrec = ntiles * 4;                      // records per replica
    const size_t nchunk = ((size_t)nrec + 255) / 256;
    for (int64_t j = 1; j <= n_sweeps; ++j) {
        const bool mj = meas && (j % measure_every) == 0;
        const float4* src = (j & 1) ? q->state : q->pingpong;
        float4* dst = (j & 1) ? q->pingpong : q->state;
        hipError_t e = xyk::launch_quad(src, dst, q->L, q->tile_x, q->tile_y, (uint32_t)q->sweep, p, mj, q->partials,
                                        q->stream);
        if (e != hipSuccess) return xyr::hip_fail(e, "xy_quad_sweep: launch");
        q->sweep += 1;
        if (mj) {
            xy_obs* rec = obs_dev + (size_t)(j / measure_every - 1) * 4;
            for (int r = 0; r < 4; ++r) {
                e = xyk::launch_finalize(q->partials + (size_t)r * nrec * 8, nrec, nullptr, rec + r, q->sweep,
                                         q->stream, q->chunks + (size_t)r * nchunk * 8, q->arrive);
                if (e != hipSuccess) return xyr::hip_fail(e, "xy_quad_sweep: finalize");
            }
        }
    }
    if (n_sweeps & 1) {                               // the last sweep wrote the second buffer
        const size_t n = (size_t)q->L * q->L;
        hipLaunchKernelGGL(xyk::k_quad_copy, dim3(2048), dim3(256), 0, q->stream, q->pingpong, q->state, n);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return xyr::hip_fail(e, "xy_quad_sweep: copy");
    }
    return XY_OK;
}

int xy_quad_set_params(xy_quad* q, const double* beta, const double* delta)
{
    if (!quad_live(q)) return XY_ESTATE;
    if (!beta || !delta) return XY_ESTATE;
    for (int r = 0; r < 4; ++r)
        if (!xyr::valid_beta_delta(beta[r], delta[r])) return XY_EINVAL;
    for (int r = 0; r < 4; ++r) {
        q->beta[r] = beta[r];
        q->delta[r] = delta[r];
    }
    return XY_OK;
}

int xy_quad_get_sweep(const xy_quad* q, uint64_t* sweep)
{
    if (!quad_live(q) || !sweep) return XY_ESTATE;
    *sweep = q->sweep;
    return XY_OK;
}

int xy_quad_set_sweep(xy_quad* q, uint64_t sweep)
{
    if (!quad_live(q)) return XY_ESTATE;
    if (sweep >= 0xffffffffull) return XY_ERANGE;
    q->sweep = sweep;
    return XY_OK;
}

int xy_quad_set_tile(xy_quad* q, int32_t tile_x, int32_t tile_y)
{
    if (!quad_live(q)) return XY_ESTATE;
    if (!xyk::quad_shape_ok(q->L, tile_x, tile_y)) return XY_EINVAL;
    q->tile_x = tile_x;
    q->tile_y = tile_y;
    q->tile_set = true;
    return XY_OK;
}

int xy_quad_get_tile(const xy_quad* q, int32_t* tile_x, int32_t* tile_y)
{
    if (!quad_live(q) || !tile_x || !tile_y) return XY_ESTATE;
    *tile_x = q->tile_x;
    *tile_y = q->tile_y;
    return XY_OK;
}

int xy_quad_hmc_work_bytes(int32_t L, size_t* bytes)
{
    if (!bytes) return XY_ESTATE;
    if (!quad_L_ok(L)) return XY_EINVAL;
    *bytes = xyk::quad_hmc_work_bytes(L);
    return XY_OK;
}

int xy_quad_hmc(xy_quad* q, int64_t n_traj, int32_t n_md, double eps, void* hmc_work, size_t hmc_len,
                xy_hmc_obs* obs_dev)
{
    if (!quad_live(q)) return XY_ESTATE;
    if (n_traj < 0 || n_md < 1 || !std::isfinite(eps) || !(eps > 0.0)) return XY_EINVAL;
    if (!hmc_work) return XY_ESTATE;
    if (hmc_len < xyk::quad_hmc_work_bytes(q->L)) return XY_ESIZE;
    if (q->sweep + (uint64_t)n_traj >= 0xffffffffull) return XY_ERANGE;
    const xyd::Params4 p = quad_params(q);
    xyk::QHmcKeys keys;
    for (int r = 0; r < 4; ++r) {
        keys.k0[r] = p.k0[r];
        keys.k1[r] = p.k1[r];
    }
    if (n_traj == 0) return XY_OK;
    const xyk::QuadHmcWork w = xyk::quad_hmc_carve(hmc_work, q->L);
    // The replicas run as four lattices: split into the second buffer at the start of
    // the call, joined into the state at its end; the state is the second angle
    // buffer of the trajectories meanwhile.  Passes as xy_hmc's default if none were
    // asked for.
    const int steps = q->hmc_steps ? q->hmc_steps : 7;
    float* planes = (float*)q->pingpong;
    hipError_t e = XY_LAUNCH(xyk::launch_quad_split(q->state, planes, q->L, q->stream));
    if (e != hipSuccess) return xyr::hip_fail(e, "xy_quad_hmc: launch");
    int rc = XY_OK;
    int64_t done = 0;
    for (; done < n_traj && rc == XY_OK;) {
        e = XY_LAUNCH(xyk::launch_quad_hmc_trajectory(planes, (float*)q->state, w, q->L, q->beta, eps, n_md, steps,
                                                      (uint32_t)q->sweep, keys,
                                                      obs_dev ? obs_dev + (size_t)done * 4 : nullptr, done > 0,
                                                      q->stream));
        if (e != hipSuccess) {
            rc = xyr::hip_fail(e, "xy_quad_hmc: launch");
        } else {
            q->sweep += 1;
            ++done;
        }
    }
    if (done > 0)
        quad_finish(rc, "xy_quad_hmc: launch",
                    [&] { return xyk::launch_quad_hmc_restore(planes, w, q->L, q->stream); });
    quad_finish(rc, "xy_quad_hmc: launch", [&] { return xyk::launch_quad_join(planes, q->state, q->L, q->stream); });
    return rc;
}

int xy_quad_hmc_set_steps_per_pass(xy_quad* q, int32_t steps)
{
    if (!quad_live(q)) return XY_ESTATE;
    if (steps < 1 || steps > kQuadHmcSteps) return XY_EINVAL;
    q->hmc_steps = steps;
    return XY_OK;
}

int xy_quad_hmc_get_steps_per_pass(const xy_quad* q, int32_t* steps)
{
    if (!quad_live(q) || !steps) return XY_ESTATE;
    *steps = q->hmc_steps ? q->hmc_steps : kQuadHmcSteps;
    return XY_OK;
}

int xy_quad_free(xy_quad* q)
{
    if (!quad_live(q)) return XY_ESTATE;
    q->magic = 0;
    delete q;
    return XY_OK;
}

}  // extern "C"
