// Internal structures shared by the host runtime (swarm_api.cpp) and the device code
// (swarm_kernels.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/swarm.h"

namespace swarm_impl {

constexpr int kMaxTraceIds = 256;
constexpr int kTallyTile = 2048;          // records per tally work-group (fixed: determinism)
constexpr int kTallyThreads = 256;
constexpr int kTally1 = 26;               // pass-1 accumulators
constexpr int kTally2 = 32;               // pass-2 accumulators
constexpr uint32_t kMaxBlocks = 0x7fffffffu;   // per-electron cap on trial blocks

// Lane states of the swarm kernels.
// ACTIVE: drawing trials; READY: holds a real-collision candidate (served with the wave's
// other READY lanes, which draw their scattering words then); IDLE: needs an electron; WAIT:
// pooled schedule, has its candidate in the work-group pool; CAND: pooled schedule, holds a
// candidate not yet in the pool; STOPPED: must store its record or state; DONE: no more work.
enum : int { ST_ACTIVE = 0, ST_IDLE = 2, ST_WAIT = 3, ST_DONE = 4, ST_STOPPED = 5, ST_READY = 6,
             ST_CAND = 7 };

// Per-channel constants built on the device from the raw inputs.
struct ChannelDev {
  int32_t kind;
  int32_t comp;
  double thr;      // threshold (eV)
  double onset;    // thr * (m+M)/M: lowest energy at which the inelastic process is allowed
  double c_ela;    // 2 m M / (m+M)^2
  double c_M;      // M / (m+M)
  double c_mM;     // (m+M) / M
  float thr_f, c_ela_f, c_M_f, c_mM_f;
  int32_t scat;    // swarm_scattering of its component
  float xi_f;
  double xi;       // SWARM_SCATTER_CONSTANT_XI: the anisotropy parameter
};

// Per-channel constants of moving targets, kept out of ChannelDev (which the kernels copy
// from LDS into registers) and read from global memory only at such collisions.
struct ThermalChannel {
  double mass;     // target mass M (kg)
  double sigma;    // sqrt(k T / M), spread of each target velocity component
  double loss;     // 2 eps_k M / ((m + M) m): the threshold in |V1 - Vcm|^2
  double cM;       // M / (m + M): V1 - Vcm = (M / (m + M)) (V1 - V2)
};

// Saved electron state at a real-collision boundary (serving epochs resume from it).
struct SavedState {
  double r[3], t;
  double v[3];
  double sum_eps, sum_epsp;
  uint64_t id;
  uint32_t block, k, k_start, G, D, n_forb, n_over, n_first;
  uint32_t started, pad;
  double nup;                 // trial frequency in use (variable strategy)
  uint32_t grace, n_fail;     // trials left before its next update; fails so far
};

// Real-secondaries runs: an electron a launch parked at a real-collision boundary (its
// resumable state and its record slot), to be resumed by the next launch together with the
// secondaries the launch created.
struct ParkedState {
  SavedState s;
  int64_t rec;
};

// At the end of a launch a wave parks only when at most park_lanes of its 64 lanes still run (by
// default kParkLanes), and at most once, so `threads` threads write at most
// parked_capacity(threads, park_lanes) states there.
constexpr int kParkLanes = 32;
constexpr int64_t parked_capacity(int64_t threads, int park_lanes) { return threads / 64 * park_lanes + 64; }

// Secondary electron in the real-secondaries queue, written by the generation that
// created it and run by the next one.
struct ChildState {
  double r[3], t;
  double v[3];
  uint64_t id;
  uint32_t k, pad;
  double eps_birth;           // energy it was created with (eV), for its first trial frequency
};

// Device counters of one instance's run.  The counters that real-mode waves update
// concurrently sit on 128-byte lines of their own, so their atomics do not queue behind
// each other.
struct RunCounters {
  uint64_t gen_next;      // electrons taken so far, of the run (real mode: of the running generation)
  uint64_t pad0[15];
  uint64_t child_tail;    // real mode: reserved secondary slots
  uint64_t pad1[15];
  uint64_t dropped;       // secondaries that did not fit the capacity
  uint64_t n_done;        // dummy mode: electrons that reached their final collision or stopped
  uint64_t parked;        // real mode: electrons the running launch parked for the next one
  uint32_t k_min;         // real mode: smallest lineage count it left to the next launch
  uint32_t pad2;
  uint64_t pad3[12];
};

// One swarm instance as seen by the kernels.  Fields in the first group are written by
// the host (pointers, sizes, run parameters); the physics constants in the second group
// are computed by the build kernels from the raw inputs.
struct InstanceDesc {
  // ---- host-written ----------------------------------------------------------------
  int32_t G, nc, p_log2, emin, emax;
  int32_t n_raw_channels;
  int32_t precision, secondaries;
  double E, B, B_angle, N, eps0, user_majorant;
  double T_K;                 // gas temperature (moving targets)
  int32_t thermal_targets;    // 1: moving targets
  int32_t relativistic;       // 1: relativistic mover (FP64, B = 0)
  int32_t trial_strategy;     // swarm_trial_strategy
  uint32_t trial_grace;       // variable and binned: trials between updates of nu'
  double trial_zeta;          // variable: nu' = (1 + zeta) nu(eps)
  int32_t trial_bins;         // binned: bins per decade
  int32_t n_bins;             // binned: number of bins (0 for the other strategies)
  const int32_t* bin_of;      // binned: bin of every entry of the padded rate table (G + 1)
  const int32_t* bin_first;   // binned: first table entry of every bin (n_bins + 1)
  const double* logtab;       // FP64 flight times: the logarithm table (unit_log.hpp)
  const double* raw_e;        // concatenated raw energies
  const double* raw_s;        // concatenated raw cross-sections
  const int32_t* raw_off;     // per channel: first point
  const int32_t* raw_n;       // per channel: number of points
  const int32_t* raw_kind;
  const int32_t* raw_comp;
  const double* raw_thr;
  const double* comp_mass_amu;
  const double* comp_frac;
  const int32_t* comp_scat;   // swarm_scattering per component
  const double* comp_ratio;   // sigma_mt / sigma_el per component
  double* nodes;              // G node energies (eV)
  double* cum_cm;             // nc x G running sums, channel major (FP64)
  double2* nu64;              // G pairs (F, F[g+1]-F[g]) of the total rate
  float2* nu32;
  double2* cum64;             // (G+1) x nc pairs, node major (row 0: below the grid), + 8 spare
  float2* cum32;
  ChannelDev* chan;
  ThermalChannel* chan_th;    // moving targets: per-channel constants (nc)
  double* bin_nup64;          // binned: nu' of every bin (built on the device)
  float* bin_nup32;
  // run parameters
  int64_t n_electrons;
  uint32_t n_collisions;
  uint32_t quantum;           // real collisions per electron per launch (0 = no limit)
  uint64_t seed;
  int64_t capacity;           // real mode: records available
  swarm_record* records;      // per-electron results
  SavedState* saved;          // resumable runs (serving); NULL otherwise
  ChildState* children;       // real mode queue
  RunCounters* ctr;
  // tracing
  const uint64_t* trace_ids;
  int32_t n_trace, max_events;
  swarm_event* trace_out;
  int32_t* trace_count;
  // ---- device-written (build kernels) ------------------------------------------------
  double majorant, inv_majorant;
  double c_eps;               // m / (2 e): eps (eV) = c_eps |v|^2
  double c_speed;             // sqrt(2 e / m): |v| = c_speed sqrt(eps)
  double speed0;
  double az;                  // -e E / m (acceleration along z)
  double omega;               // e B / m
  double bx, bz;              // unit vector of B
  double vDy;                 // E x B / B^2 = (0, E sin(th) / B, 0)
  double apar;                // a . b
  double numax;
  float majorant_f, cT_f;     // cT_f = ln2 / nu' (flight time from log2)
  float c_eps_f, c_speed_f, speed0_f, az_f, omega_rev_f, bx_f, bz_f, vDy_f, apar_f;
  float sceps_f, aze_f, apare_f, nup24_f, Pf_f, twoPf_f;   // FP32 energy-unit constants
  double Pf_d, twoPf_d;
  double rel_kEc, rel_kBx, rel_kBz;       // relativistic mover in E and B: generator and
  double rel_l1, rel_l2, rel_p1, rel_p2, rel_K;   // field invariants
  int32_t built_ok;           // 1 after a successful build, -1 if a node has zero rate
  // Lowest node at which an electron of that energy loses at least what the field gives it
  // (the host sets it to the top node, the build lowers it), and the trials per real collision
  // there.  They shape launches only; no result depends on them.
  uint32_t balance_node;
  int32_t trigger;            // waiting lanes of a full wave at which it serves them, by default
  double trials;
};

// How many electrons a wave takes at a time when `left` are left (as far as it knows) and its
// idle lanes want `wanted`: `chunk` while more than `scarce` are left, then `share` of what is
// left, and never fewer than it wants.  Every claim is an atomic on the launch's one counter
// that the wave waits for.  The generations of a real-secondaries run take shares: with only what
// their lanes wanted (share 0) from two chunks per wave on, a generation of two or three
// rounds made a claim for nearly every electron (FP32, wanted only | shares, ms: 1e6 primaries x 300
// in argon at 30 Td 10.4 | 9.5, in Ar:CO2 at 100 Td 19.2 | 16.6; 1e6 x 100 in argon at 100 Td 9.0 |
// 7.5; 1e5 x 2000 of the magnetised mixture 64.5 | 61.4).  Dummy launches take what they want: they
// end on finer steps that way (argon sweep 32 x 1e5 x 2e4 FP32 727 ms, with shares 733; FP64 of one
// magnetised mixture, 4e5 x 500, 11.4 | 13.1), and electrons that end often are held up by
// their count in RunCounters::n_done sooner than by claims.
struct ClaimRule {
  uint32_t chunk = 1, scarce = 0;
  float share = 0.0f;
  __host__ __device__ uint32_t size(uint32_t left, uint32_t wanted) const {
    if (left > scarce) return chunk;
    const uint32_t n = static_cast<uint32_t>(static_cast<float>(left) * share);
    return n > wanted ? n : wanted;
  }
};
// From `chunks` more claims of every wave on: no more than its idle lanes want, or with
// `shares` a part of an even share of what is left (a `chunks`-th of it, so that the sizes go
// on from the chunk).
inline ClaimRule claim_rule(uint32_t chunk, int64_t waves, int chunks, bool shares) {
  ClaimRule r;
  const uint64_t all = static_cast<uint64_t>(chunks) * static_cast<uint64_t>(waves);
  const uint64_t scarce = all * chunk;
  r.chunk = chunk;
  r.scarce = scarce < 0xffffffffull ? static_cast<uint32_t>(scarce) : 0xffffffffu;
  r.share = shares ? 1.0f / static_cast<float>(all) : 0.0f;
  return r;
}

// Slices of the lineage budget in a real-secondaries run.  A generation by itself lasts as long
// as its longest electron, so while few electrons are left a run would spend its time on a few
// long chains, generation after generation.  A launch of few electrons therefore runs them only
// up to a common lineage count, parks them there, and the next launch resumes them together with
// the secondaries, which have caught up by its end.  That holds from the start while the run is
// small (for the device's `lanes`, four waves per SIMD), and again once the generations have
// shrunk, from the smallest lineage count left.
// A slice costs a launch and a wait for its slowest electron (20,000 electrons that ionise
// nothing, FP32: 0.4 ms for 128 collisions that take 0.5), and it gains nothing where no
// generation follows.  A gas without ionisation is never sliced.  A slice is doubled while fewer
// than a hundredth of its electrons (of the few that do not fill a wave per SIMD, for which
// slices cost less, a four-hundredth) ionise in it, both in the last one and by the rate
// counted so far, and it is short again when a twenty-fifth do in one.  The count stands for a
// quarter more than it says, as few electrons count nothing for a while: with one more, 25 argon
// electrons waited sixteen slices for the first doubling (FP32 ms, one more and a quarter more, 50
// x 3000 at 3 Td 8.0 and 7.0, adaptive at 10 Td 7.1 and 6.5, the mixture at 20 Td 7.9 and 8.5; over
// 176 runs of 25 to 1000 electrons 3% faster).
struct SlicePlan {
  int64_t budget, lanes, room;      // collisions of a lineage; parked electrons that fit
  bool ionises;                     // the gas has an ionisation channel (and parking is allowed)
  int64_t reached = 0;              // lineage count that the electrons of the next launch have reached
  int64_t length = 0;               // of a slice, 0: the shortest
  bool growing = true;              // no launch has run whole generations yet
  bool sliced = false;              // the launch under way
  double born = 0.0, work = 0.0;    // secondaries and electron-collisions counted at `length` or below
  // The lineage count at which a launch of `electrons` parks them.
  int64_t limit(int64_t electrons) {
    sliced = ionises && electrons <= room && electrons <= (growing ? lanes / 8 : lanes / 8 * 3);
    growing = growing && sliced;
    if (!sliced || length == 0) length = 0, born = work = 0.0;
    length = std::max<int64_t>(length, electrons <= lanes / 64 ? 64 : 128);
    return sliced && budget - reached > length ? reached + length : budget;
  }
  // What that launch did: secondaries made, smallest lineage count left.
  void launched(int64_t electrons, int64_t made, int64_t at, int64_t smallest) {
    reached = sliced ? at : smallest;
    if (!sliced) return;
    born += static_cast<double>(made);
    work += static_cast<double>(electrons) * static_cast<double>(length);
    const int64_t few = electrons <= lanes / 64 ? 400 : 100;
    if (made * 25 > electrons) length = 0;
    else if (made * few < electrons && (born + 0.25) * static_cast<double>(few * length) < work && length < budget) length *= 2;
  }
};

// How a launch hands out the electrons of its instances.  Every instance has a line of 64 bytes
// with the number of those taken and, behind it, of the work-groups that came to it; a wave takes
// some electrons at a time and passes them to its lanes.  A work-group starts with instance
// first[blockIdx.x] (NULL: instance 0), stays with it until all of its electrons are taken and
// run, and goes on with an instance that has much work left for the work-groups on it: weight
// (expected work per electron) times electrons not taken (next_instance).
constexpr int kClaimStride = 8;           // counters are this many 64-bit words apart
struct ClaimPlan {
  unsigned long long* taken;
  const int32_t* first;
  const float* weight;
  const uint32_t* count;                  // electrons per instance
  int32_t n_inst;
  int32_t chunk;                          // the rule's chunk (launches of teams set their own)
  ClaimRule rule = {};
};

struct TallyTile {
  int32_t inst;
  int32_t tile;        // tile index within the instance
  int64_t first;
  int64_t count;
};

// Launch shape of the team kernels: `lanes` lanes per electron (a power of two up to 32; 1: the
// one-lane kernels, and the other fields are not used), `per_wave` teams in every wave (its
// other lanes stay idle), work-groups of `block`, and the waiting lanes, in 64ths of a wave's
// running ones, at which it serves collisions.
struct TeamShape {
  int lanes = 1, per_wave = 64, block = 64, trigger = 48;
  int64_t per_group() const { return static_cast<int64_t>(per_wave) * (block / 64); }   // electrons at once
};

// Launchers implemented in swarm_kernels.hip.
hipError_t launch_build(InstanceDesc* d_desc, const InstanceDesc& h_desc, hipStream_t s);
hipError_t launch_fill_u32(uint32_t* p, uint32_t v, int64_t n, hipStream_t s);
hipError_t launch_mark_empty(swarm_record* r, int64_t n, hipStream_t s);
hipError_t launch_fill_u64(uint64_t* p, uint64_t v, int64_t n, hipStream_t s);
// pending_trigger 0: every instance's own.  service_waves > 0 (and no trace): the pooled schedule, pool at LDS offset pool_off.
hipError_t launch_swarm_dummy(const InstanceDesc* d_desc, ClaimPlan plan, int precision, bool has_b, bool trace,
                              int ext, int service_waves, int block_size, int grid, int pending_trigger,
                              size_t lds_bytes, int ch_off, int pool_off, int cum_off, hipStream_t s,
                              TeamShape team);
size_t swarm_pool_slot_bytes(int precision);
// One real-secondaries launch: the n_park_in electrons in park_in (parked by the launch
// before), then `count` electrons from `first` (the primaries if first < 0, else queued
// secondaries).  An electron whose lineage count reaches k_limit, or slice collisions more than
// it starts with if that is later, before its budget's end is parked in park_out (park_cap
// slots; past them it runs on).  Once every electron is claimed, a
// wave left with few running lanes parks them too, at their next real-collision boundary,
// provided this launch has created at least park_min secondaries (the queue started at tail0);
// park_lanes is the most running lanes such a wave may have, and park_min <= 0 parks none this
// way.  The next launch runs the parked electrons together with the secondaries.
hipError_t launch_swarm_real(const InstanceDesc* d_desc, int precision, bool has_b, bool trace,
                             int ext, int block_size, int grid, int pending_trigger, size_t lds_bytes,
                             int ch_off, int cum_off, int64_t first, int64_t count, int flush,
                             const ParkedState* park_in, int64_t n_park_in, ParkedState* park_out,
                             int64_t park_min, int park_lanes, int64_t tail0, uint32_t k_limit, uint32_t slice, int64_t park_cap, hipStream_t s,
                             TeamShape team);
// Resets the counters of a real-secondaries launch (electrons taken and parked, smallest count).
hipError_t launch_next_generation(RunCounters* ctr, hipStream_t s);
hipError_t launch_tallies(const InstanceDesc* d_desc, const TallyTile* d_tiles, int32_t n_tiles,
                          const int32_t* d_tile_base, const int64_t* d_nrec, int32_t n_inst,
                          double* d_part1, double* d_part2, double* d_tot1,
                          swarm_tallies_t* d_out, hipStream_t s);
int swarm_kernel_max_blocks_per_cu(int precision, bool has_b, bool trace, bool real, int ext,
                                   int service_waves, int block_size,
                                   size_t lds_bytes, bool team = false);

}  // namespace swarm_impl
