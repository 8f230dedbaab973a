// xy_launch.hpp -- host-side launchers of the HIP kernels (internal to the library).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "xy.h"

namespace xyd {
struct Params4;       // xy_tile4.hpp
}

namespace xyk {

struct SweepArgs {
    void* src;          // state read by the sweep
    void* dst;          // state written (== src for in-place schedules)
    int L;
    int precision;      // XY_FP32 / XY_FP16
    uint32_t key0, key1;
    uint32_t sweep;     // absolute index of the (first) sweep
    float delta, nbl2e;   // proposal width in turns (FP32), -beta log2(e)
};

// Workspace carve-up shared by the runtime and the launchers.
struct Work {
    void* pingpong;                 // second state buffer (fused schedule)
    unsigned long long* counter;    // accept counter (one u64)
    unsigned* arrive;               // arrival counter of the one-launch finalize (zeroed with counter)
    double* partials;               // per-workgroup measurement partials, 8 doubles each
    int max_partials;
    double* chunks;                 // second-level sums of 256 partials each
};

size_t state_bytes(int L, int precision);
size_t work_bytes(int L, int precision);
Work carve(void* work, int L, int precision);
int max_partials_for(int L);

hipError_t launch_init(void* st, int L, int precision, uint32_t k0, uint32_t k1, int hot, hipStream_t s);

// One half-sweep of `colour`, in place.  counter != NULL adds the accepts to it;
// dbg_acc / dbg_dE != NULL write per-site decisions and FP32 dE in the state layout.
hipError_t launch_half_sweep(const SweepArgs& a, int colour, unsigned long long* counter,
                             uint8_t* dbg_acc, float* dbg_dE, hipStream_t s);

// FP64 partial sums of the observables of state `st` into partials[0..*nparts).
hipError_t launch_measure(const void* st, int L, int precision, double* partials, int max_parts,
                          int* nparts, hipStream_t s);

// Reduce partials in a fixed order, take the accept counter (and clear it) plus the
// accepts in slot 6 of the partials, write one xy_obs record.  More than 2048
// partials take two levels in one launch, through `chunks` (the sums of 256 partials
// each) and `arrive` (a zeroed u32 in device memory, zero again afterwards).
hipError_t launch_finalize(const double* partials, int nparts, unsigned long long* counter,
                           xy_obs* out, uint64_t sweep_after, hipStream_t s, double* chunks, unsigned* arrive);

// Fused tiled sweep(s): `m` sweeps (1 or 2) per launch from a.src to a.dst.
// meas_mask bit j set: measure after sub-sweep j into the 8-double record
// partials[(j * ntiles + tile) * 8] (slot 6 = the tile's accepts).
hipError_t launch_fused(const SweepArgs& a, int tile_x, int tile_y, int m, unsigned meas_mask,
                        double* partials, hipStream_t s);
int fused_tiles(int L, int tile_x, int tile_y);
// One sweep by tiles of tile_x (128 or 256) x 16 sites that need not divide the
// lattice; measured: ragged_records(L, tile_x) partial records, their terms
// gathered as launch_measure does.
int ragged_tile_x(int L);        // the faster width, 0 if the lattice is out of range
int ragged_records(int L, int tile_x);
hipError_t launch_ragged(const SweepArgs& a, int tile_x, bool meas, double* partials, hipStream_t s);
// One sweep by strips of one wave (xy_walk.hip); measured: walk_records(L) partial
// records.
bool walk_supported(int L, int precision, bool meas);
int walk_records(int L);
hipError_t launch_walk(const SweepArgs& a, bool meas, double* partials, hipStream_t s);
// An unmeasured sweep of the four lattices of a quad.
bool walk_quad_supported(int L);
hipError_t launch_walk_quad(const float* src, float* dst, int L, uint32_t sweep, const xyd::Params4& p, hipStream_t s);
// Partial records one measured sweep of a fused launch writes (the sweep's
// records start at partials + j * fused_records(...) * 8 for sub-sweep j).
int fused_records(int L, int tile_x, int tile_y, int m);

// Strip sweep (xy_strip.hip): one sweep from a.src to a.dst by segments of
// tile_x columns x tile_y rows; measured: one record per wave (4 per segment) at
// partials[(segment * 4 + wave) * 8].
bool strip_supported(int L, int tile_x, int tile_y);
// Whole lattice resident in one workgroup's LDS (L <= 128, L % 4 == 0): n sweeps
// in place from a.src (= a.dst), records of every me-th sweep of the call to
// obs[0 ..] (none if me == 0 or obs == NULL).
bool resident_supported(int L);
hipError_t launch_resident(const SweepArgs& a, int n, int me, xy_obs* obs, hipStream_t s);
// The same for any even L <= 62, the records' terms gathered as launch_measure does.
hipError_t launch_resident_any(const SweepArgs& a, int n, int me, xy_obs* obs, hipStream_t s);
hipError_t launch_strip(const SweepArgs& a, int tile_x, int tile_y, bool meas, double* partials, hipStream_t s);
int strip_records(int L, int tile_x, int tile_y);

// Several sweeps per launch (xy_deep.hip): the lattice cut into tx x ty regions,
// each grown so that n sweeps need no other region's results.
struct DeepPlan {
    int tx, ty;           // cores along a row and down the lattice
    int PC, RY, hx, hy;   // a region's pairs and rows, its halo in pairs and rows
    int rp, full;         // measured: columns of `full` pairs `rp` rows apart (0: pair by pair)
};
// The regions of d's tx x ty cores for n sweeps, if they fit into the lattice.
bool deep_region(int L, int n, DeepPlan* d);
// The regions and the most sweeps per launch for lattices and calls of n sweeps
// that gain from it; `meas`: for passes with a measured sweep.
bool deep_choose(int L, int64_t n, bool meas, DeepPlan* d, int* nmax);
// n sweeps from a.src to a.dst (two buffers).  Sweep j (1-based) is measured when
// me > 0 and (j + phase) % me == 0, phase < me; the k-th measured one leaves a record of
// region b at part[(k * tx * ty + b) * 8].
hipError_t launch_deep(const SweepArgs& a, const DeepPlan& d, int n, int me, int phase, double* part, hipStream_t s);
// nrec records of np partial records each, back to back in `part`, into out[0 ..];
// record k's sweep count is first + (k / group) * every.
hipError_t launch_finalize_many(const double* part, int np, int nrec, xy_obs* out, uint64_t first, int every,
                                hipStream_t s, int group = 1);

// ---- hybrid Monte Carlo (xy_hmc.hip)
constexpr int kHmcMaxRecords = 65536;   // partial records of one H sum (old or new)
constexpr int kHmcMaxChunks = kHmcMaxRecords / 256;
struct HmcWork {
    unsigned* flag;     // accept flag of the last trajectory
    float* p;           // momenta, state layout
    float* saved;       // angles at the start of the trajectory
    float* p2;          // second momentum buffer (passes of several steps)
    double* rec_old;    // partial records of H_old (8 doubles each)
    double* rec_new;    // partial records of H_new
    double* chunk_old;  // sums of 256 records each
    double* chunk_new;
};
size_t hmc_work_bytes(int L);
HmcWork hmc_carve(void* work, int L);
int hmc_records(int L);
// One trajectory from the FP32 angles in `state` (result back in `state`),
// `pingpong` a second state-sized buffer; record to obs if not NULL.
// again: another trajectory of the same call went before, and no restore since.
// steps_per_pass > 1: leap-frog steps in passes of up to min(steps_per_pass, 8)
// steps (temporal blocking); else one step per launch.
hipError_t launch_hmc_trajectory(float* state, float* pingpong, const HmcWork& w, int L, double beta, double eps,
                                 int n_md, int steps_per_pass, uint32_t traj, uint32_t k0, uint32_t k1,
                                 xy_hmc_obs* obs, bool again, hipStream_t s);
// After the last trajectory of a call: the saved angles back into the state if it
// was rejected.
hipError_t launch_hmc_restore(float* state, const HmcWork& w, int L, hipStream_t s);
// Workspace of one lattice with record arrays sized for its L only (batches).
size_t hmc_work_bytes_compact(int L);
HmcWork hmc_carve_compact(void* work, int L);

// One trajectory of many lattices, one launch per stage over all of them
// (batches).  Lattice i's numbers and arithmetic are those of
// launch_hmc_trajectory on it alone, so each lattice is bit for bit the
// single-lattice trajectory.  L % 4 == 0.
struct BhLat {
    float* st;          // the lattice's angles
    float* pp;          // its second angle buffer
    HmcWork w;          // its HMC areas (hmc_carve_compact)
    xy_hmc_obs* obs;    // where its trajectory record goes (may be NULL)
    double beta;
    int L, cols, rb, nrec;        // rb: row runs of the pair kernels (hmc_runs2)
    uint32_t k0, k1;
    float kick_half, kick_full;   // -beta eps / 2, -beta eps (FP32, as launch_hmc_trajectory forms them)
};
// Fill the geometry fields of d (cols, rb, nrec, kicks) for lattice L at beta, eps.
void hmc_batch_describe(BhLat& d, int L, double beta, double eps);
// Leap-frog steps of the longest pass, and the rows a thread takes in the passes (0:
// one step a launch, not in regions).
int hmc_batch_steps(int n_md, int steps_per_pass);
int hmc_batch_rows(int n, const int32_t* L, int kh);
// Workgroups lattice L takes in each stage grid: [0] ends, [1] leap-frog pass of kh
// steps, [2] restore (each a multiple of 8, so that every lattice starts on XCD 0).
void hmc_batch_blocks(int L, int rows, int kh, uint32_t nb[3]);
// d: n descriptors in device memory; start: 3 (n + 1) block offsets in device
// memory (stage s, lattice i at start[s (n + 1) + i], each stage's total last),
// totals the three grid sizes; traj_dev: the trajectory index in device memory.
hipError_t launch_hmc_batch_trajectory(const BhLat* d, const uint32_t* start, int n, const uint32_t totals[3],
                                       double eps, int n_md, int steps_per_pass, int rows, const uint32_t* traj_dev,
                                       hipStream_t s);
bool fused_supported(int L, int tile_x, int tile_y, int m);

// ---- sweeps of the four replicas of a quad
// Several sweeps per launch as launch_deep, from one float4 state to another; the
// k-th measured sweep leaves a record of replica r, region b at
// part[((4 k + r) * tx * ty + b) * 8].
bool deep_choose_quad(int L, int64_t n, DeepPlan* d, int* nmax);
hipError_t launch_deep_quad(const float4* src, float4* dst, int L, uint32_t sweep, const xyd::Params4& p,
                            const DeepPlan& d, int n, int me, int phase, double* part, hipStream_t s);
// The whole quad in four workgroups (L <= 32): n sweeps in place, records of every
// me-th one to obs[0 .. 3], obs[4 .. 7] ... (none if me == 0 or obs == NULL).
hipError_t launch_resident_quad(float4* state, int L, uint32_t sweep, const xyd::Params4& p, int n, int me, xy_obs* obs,
                                hipStream_t s);
// The four records of one sweep, replica r's from the nrec partial records at
// partials + r * nrec * 8, through `chunks` (4 * ceil(nrec / 256) records) and the
// arrival counters arrive[0 .. 3].
hipError_t launch_finalize_quad(const double* partials, int nrec, xy_obs* out, uint64_t sweep_after, double* chunks,
                                unsigned* arrive, hipStream_t s);

// ---- the four replicas of a quad as four lattices back to back
struct QHmcKeys {
    uint32_t k0[4], k1[4];        // Philox keys of the four replicas
};
struct QHmcBeta {
    double b[4];
};
// The float4 state's components into four lattices of L^2 floats each, and back.
hipError_t launch_quad_split(const float4* state, float* planes, int L, hipStream_t s);
hipError_t launch_quad_join(const float* planes, float4* state, int L, hipStream_t s);

// ---- hybrid Monte Carlo on them (xy_hmc.hip)
struct QuadHmcWork {
    float* p;           // momenta, as the lattices
    float* saved;       // angles at the start of the trajectory
    float* p2;          // second momentum buffer
    unsigned* flag;     // per replica (16 words apart) the last decision and an arrival counter
    double* rec_old;    // partial records of H_old: replica r's at rec_old + r * records * 8
    double* rec_new;
    double* chunk_old;  // sums of 256 records each, per replica
    double* chunk_new;
};
size_t quad_hmc_work_bytes(int L);
QuadHmcWork quad_hmc_carve(void* work, int L);
// One trajectory of all four replicas, each bit for bit launch_hmc_trajectory's of
// its lattice (its FP64 sums may be cut differently); obs: NULL or 4 records.
hipError_t launch_quad_hmc_trajectory(float* planes, float* second, const QuadHmcWork& w, int L, const double beta[4],
                                      double eps, int n_md, int steps_per_pass, uint32_t traj, const QHmcKeys& keys,
                                      xy_hmc_obs* obs, bool again, hipStream_t s);
hipError_t launch_quad_hmc_restore(float* planes, const QuadHmcWork& w, int L, hipStream_t s);

// Fill n u64 words with zero (kernel, not a memset node: safe inside graphs).
hipError_t launch_zero_u64(unsigned long long* p, int n, hipStream_t s);

}  // namespace xyk
