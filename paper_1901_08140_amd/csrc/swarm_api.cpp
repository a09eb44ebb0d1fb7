// Host runtime of libswarm: argument validation, device memory, kernel launches, hipGraph
// capture of batched launches, the launch-shape autotuner and the C ABI of swarm.h.
// No method arithmetic happens here: tables, physics constants, the simulation and the
// tallies are all computed by the kernels in swarm_kernels.hip.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <memory>
#include <string>
#include <vector>

#include "swarm_api_internal.hpp"
#include "unit_log.hpp"

using namespace swarm_impl;

namespace swarm_impl {

thread_local std::string g_last_error;

swarm_status fail(swarm_status st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return st;
}

swarm_status hip_fail(hipError_t e, const char* what) {
  return fail(e == hipErrorOutOfMemory ? SWARM_ERR_OUT_OF_MEMORY : SWARM_ERR_DEVICE, "%s: %s", what,
              hipGetErrorString(e));
}

DeviceInfo& device_info() {
  static DeviceInfo info = [] {
    DeviceInfo d{};
    if (hipGetDevice(&d.device) != hipSuccess) d.device = 0;
    hipDeviceProp_t p;
    if (hipGetDeviceProperties(&p, d.device) == hipSuccess) {
      d.n_cu = p.multiProcessorCount;
      d.lds_per_block = static_cast<int64_t>(p.sharedMemPerBlock);
    } else {
      d.n_cu = 256;
      d.lds_per_block = 65536;
    }
    return d;
  }();
  return info;
}

// Dynamic LDS of the swarm kernels: the total-rate pairs of the G grid nodes plus one
// padding entry in front, then (16-byte aligned) the nc channel descriptors, then with table
// layout 1 the (G+1) x nc running-sum pairs (if everything fits the work-group's LDS), then with
// the pooled schedule the candidate pool (64 slots per service wave).
LdsLayout lds_layout(int precision, int G, int nc, int service_waves, int table_layout) {
  auto al = [](size_t n) { return (n + 15) & ~static_cast<size_t>(15); };
  const size_t pair = precision == SWARM_FP32_MIXED ? sizeof(float2) : sizeof(double2);
  const size_t pool = service_waves > 0 ? static_cast<size_t>(64 * service_waves) * swarm_pool_slot_bytes(precision) : 0;
  LdsLayout l;
  l.ch_off = static_cast<int>(al(static_cast<size_t>(G + 1) * pair));
  const size_t after_ch = al(static_cast<size_t>(l.ch_off) + static_cast<size_t>(nc) * sizeof(ChannelDev));
  l.cum_off = -1;
  l.pool_off = static_cast<int>(after_ch);
  if (table_layout == 1) {
    const size_t with_cum = al(after_ch + (static_cast<size_t>(G + 1) * static_cast<size_t>(nc) + 8) * pair);
    if (static_cast<int64_t>(with_cum + pool) <= device_info().lds_per_block) {
      l.cum_off = static_cast<int>(after_ch);
      l.pool_off = static_cast<int>(with_cum);
    }
  }
  l.bytes = static_cast<size_t>(l.pool_off) + pool;
  return l;
}

constexpr size_t kArenaAlign = 256;

Arena::Arena(void* base, size_t bytes) {
  const uintptr_t b = reinterpret_cast<uintptr_t>(base);
  const uintptr_t a = (b + kArenaAlign - 1) & ~static_cast<uintptr_t>(kArenaAlign - 1);
  const size_t lost = static_cast<size_t>(a - b);
  base_ = reinterpret_cast<char*>(a);
  bytes_ = bytes > lost ? ((bytes - lost) & ~(kArenaAlign - 1)) : 0;
  if (bytes_ > 0) free_[0] = bytes_;
}

void* Arena::alloc(size_t n) {
  const size_t want = std::max(kArenaAlign, (n + kArenaAlign - 1) & ~(kArenaAlign - 1));
  std::lock_guard<std::mutex> lk(mu_);
  for (auto it = free_.begin(); it != free_.end(); ++it) {
    if (it->second < want) continue;
    const size_t off = it->first, size = it->second;
    free_.erase(it);
    if (size > want) free_[off + want] = size - want;
    used_[off] = want;
    in_use_ += want;
    return base_ + off;
  }
  return nullptr;
}

void Arena::release(void* p) {
  if (!p) return;
  std::lock_guard<std::mutex> lk(mu_);
  auto u = used_.find(static_cast<size_t>(static_cast<char*>(p) - base_));
  if (u == used_.end()) return;
  size_t off = u->first, size = u->second;
  used_.erase(u);
  in_use_ -= size;
  auto next = free_.lower_bound(off);
  if (next != free_.end() && off + size == next->first) {   // merge with the block after
    size += next->second;
    next = free_.erase(next);
  }
  if (next != free_.begin()) {                               // and with the block before
    auto prev = std::prev(next);
    if (prev->first + prev->second == off) {
      prev->second += size;
      return;
    }
  }
  free_[off] = size;
}

size_t Arena::in_use() const {
  std::lock_guard<std::mutex> lk(mu_);
  return in_use_;
}

DevBuf::~DevBuf() { reset(); }
void DevBuf::reset() {
  if (p) {
    if (arena) arena->release(p);
    else (void)hipFree(p);
  }
  p = nullptr;
  bytes = 0;
}
hipError_t DevBuf::ensure(size_t n) {
  if (n <= bytes && p) return hipSuccess;
  reset();
  if (n == 0) return hipSuccess;
  if (arena) {
    p = arena->alloc(n);
    if (!p) return hipErrorOutOfMemory;
  } else {
    hipError_t e = hipMalloc(&p, n);
    if (e != hipSuccess) {
      p = nullptr;
      return e;
    }
  }
  bytes = n;
  return hipSuccess;
}

size_t tally_bytes(int64_t n_records) {
  auto blk = [](size_t n) { return std::max(kArenaAlign, (n + kArenaAlign - 1) & ~(kArenaAlign - 1)); };
  const size_t tiles = static_cast<size_t>(std::max<int64_t>(1, (n_records + kTallyTile - 1) / kTallyTile));
  return blk(tiles * sizeof(TallyTile)) + blk(sizeof(int32_t)) + blk(sizeof(int64_t)) +
         blk(tiles * kTally1 * sizeof(double)) + blk(tiles * kTally2 * sizeof(double)) +
         blk((kTally1 + kTally2) * sizeof(double)) + blk(sizeof(swarm_tallies_t));
}

}  // namespace swarm_impl

namespace {

// Bins of the binned trial frequency (BinnedTrialFrequency, section "Trial frequency
// strategies"): b per decade of energy, bin k = [10^(k/b), 10^((k+1)/b)) eV, counted from the
// bin of the lowest grid node.  A grid cell belongs to the bin of its lower node.  The table
// is indexed like the padded rate table of the kernels: entry 0 (below the grid) belongs to
// node 0, entry g + 1 to node g (its cell, or for the top node the energies above it).
// Bins are numbered from 0 to the top node's bin; on a coarse grid some hold no node (their
// nu' is 0 and only the range maximum after a fail visits them).  Entries first[k] ..
// first[k+1] - 1 are those of bin k (an empty range for an empty bin); first[n_bins] = G + 1.
// Node energies are exact (a power of two times 1 + i/P); 1, 10, 100 and 1000 eV are nodes,
// and log10 returns their exact logarithms, so those nodes open their bins.
void decade_bins(int P, int emin, int G, int b, std::vector<int32_t>& entry_bin, std::vector<int32_t>& first) {
  auto bin = [&](int g) {
    const double e = std::ldexp(1.0 + static_cast<double>(g % P) / P, emin + g / P);
    return static_cast<int32_t>(std::floor(std::log10(e) * b));
  };
  const int32_t k0 = bin(0);
  entry_bin.assign(G + 1, 0);
  for (int i = 1; i <= G; ++i) entry_bin[i] = bin(i - 1) - k0;
  const int nb = entry_bin[G] + 1;
  first.assign(nb + 1, G + 1);
  for (int i = G; i >= 0; --i) first[entry_bin[i]] = i;
  for (int k = nb - 1; k >= 0; --k) first[k] = std::min(first[k], first[k + 1]);
}

swarm_status busy() {
  return fail(SWARM_ERR_STATE, "a run started by swarm_run_async is in flight: call swarm_wait first");
}

swarm_status validate(const swarm_component* comps, int32_t n_comps, const swarm_params* p) {
  if (!comps || n_comps <= 0) return fail(SWARM_ERR_INVALID_ARG, "need at least one component");
  if (!p) return fail(SWARM_ERR_INVALID_ARG, "params is NULL");
  if (!(p->N_per_m3 > 0.0) || !std::isfinite(p->N_per_m3)) return fail(SWARM_ERR_INVALID_ARG, "N must be > 0");
  if (!(p->E_V_per_m >= 0.0) || !std::isfinite(p->E_V_per_m)) return fail(SWARM_ERR_INVALID_ARG, "E must be >= 0");
  if (!(p->B_T >= 0.0) || !std::isfinite(p->B_T)) return fail(SWARM_ERR_INVALID_ARG, "B must be >= 0");
  if (!std::isfinite(p->B_angle_rad)) return fail(SWARM_ERR_INVALID_ARG, "B angle must be finite");
  if (!(p->init_energy_eV >= 0.0) || !std::isfinite(p->init_energy_eV))
    return fail(SWARM_ERR_INVALID_ARG, "initial energy must be >= 0");
  if (p->precision != SWARM_FP64 && p->precision != SWARM_FP32_MIXED)
    return fail(SWARM_ERR_INVALID_ARG, "unknown precision %d", p->precision);
  if (p->secondaries != SWARM_DUMMY && p->secondaries != SWARM_REAL)
    return fail(SWARM_ERR_INVALID_ARG, "unknown secondaries mode %d", p->secondaries);
  if (!(p->user_majorant >= 0.0) || !std::isfinite(p->user_majorant))
    return fail(SWARM_ERR_INVALID_ARG, "user majorant must be >= 0");
  if (p->capacity < 0) return fail(SWARM_ERR_INVALID_ARG, "capacity must be >= 0");
  if (p->trial_strategy != SWARM_TRIAL_CONSTANT && p->trial_strategy != SWARM_TRIAL_VARIABLE &&
      p->trial_strategy != SWARM_TRIAL_BINNED)
    return fail(SWARM_ERR_INVALID_ARG, "unknown trial strategy %d", p->trial_strategy);
  if (p->trial_strategy == SWARM_TRIAL_VARIABLE) {
    if (!(p->trial_zeta >= 0.0) || !std::isfinite(p->trial_zeta))
      return fail(SWARM_ERR_INVALID_ARG, "trial zeta must be finite and > 0 (0 = default)");
  }
  if (p->trial_strategy != SWARM_TRIAL_CONSTANT && (p->trial_grace < 0 || p->trial_grace > 0x7fffffffLL))
    return fail(SWARM_ERR_INVALID_ARG, "trial grace must be in [1, 2^31 - 1] (0 = default)");
  if (p->trial_strategy == SWARM_TRIAL_BINNED && (p->trial_bins < 0 || p->trial_bins > 100))
    return fail(SWARM_ERR_INVALID_ARG, "trial bins per decade must be in [1, 100] (0 = default)");
  if (p->thermal_targets != 0 && p->thermal_targets != 1)
    return fail(SWARM_ERR_INVALID_ARG, "thermal_targets must be 0 or 1");
  if (p->thermal_targets && (!(p->T_K >= 0.0) || !std::isfinite(p->T_K)))
    return fail(SWARM_ERR_INVALID_ARG, "moving targets need a gas temperature T_K >= 0");
  if (p->relativistic != 0 && p->relativistic != 1) return fail(SWARM_ERR_INVALID_ARG, "relativistic must be 0 or 1");
  if (p->relativistic && p->thermal_targets)
    return fail(SWARM_ERR_INVALID_ARG, "the relativistic mover does not take moving targets");
  if (p->relativistic && p->precision != SWARM_FP64)
    return fail(SWARM_ERR_INVALID_ARG, "the relativistic mover runs in SWARM_FP64");
  const int P = p->grid_points_per_octave ? p->grid_points_per_octave : 64;
  if (P <= 0 || P > 1024 || (P & (P - 1)) != 0)
    return fail(SWARM_ERR_INVALID_ARG, "grid points per octave must be a power of two <= 1024");
  int emin = p->grid_min_exp2, emax = p->grid_max_exp2;
  if (emin == 0 && emax == 0) { emin = -14; emax = 12; }
  if (emax <= emin || emin < -60 || emax > 60) return fail(SWARM_ERR_INVALID_ARG, "bad grid exponent range");
  double fsum = 0.0;
  int nc = 0;
  for (int k = 0; k < n_comps; ++k) {
    const swarm_component& c = comps[k];
    if (!(c.mass_amu > 0.0) || !std::isfinite(c.mass_amu))
      return fail(SWARM_ERR_INVALID_ARG, "component %d: mass must be > 0", k);
    if (!(c.fraction >= 0.0) || !std::isfinite(c.fraction))
      return fail(SWARM_ERR_INVALID_ARG, "component %d: fraction must be >= 0", k);
    if (c.n_channels <= 0 || !c.channels) return fail(SWARM_ERR_INVALID_ARG, "component %d: no channels", k);
    if (c.scattering < SWARM_SCATTER_ISOTROPIC || c.scattering > SWARM_SCATTER_CONSTANT_XI)
      return fail(SWARM_ERR_INVALID_ARG, "component %d: unknown scattering %d", k, c.scattering);
    if (c.scattering == SWARM_SCATTER_CONSTANT_XI && !(c.mt_over_el > 0.0 && c.mt_over_el <= 1.0))
      return fail(SWARM_ERR_INVALID_ARG, "component %d: sigma_mt/sigma_el must be in (0, 1]", k);
    fsum += c.fraction;
    for (int j = 0; j < c.n_channels; ++j) {
      const swarm_channel& q = c.channels[j];
      if (q.kind < 0 || q.kind > 3) return fail(SWARM_ERR_INVALID_ARG, "component %d channel %d: bad kind", k, j);
      if (!(q.threshold_eV >= 0.0) || !std::isfinite(q.threshold_eV))
        return fail(SWARM_ERR_INVALID_ARG, "component %d channel %d: threshold must be >= 0", k, j);
      if (q.n_points < 2 || !q.energy_eV || !q.sigma_m2)
        return fail(SWARM_ERR_INVALID_ARG, "component %d channel %d: need >= 2 points", k, j);
      for (int i = 0; i < q.n_points; ++i) {
        if (!(q.energy_eV[i] > 0.0) || !std::isfinite(q.energy_eV[i]))
          return fail(SWARM_ERR_INVALID_ARG, "component %d channel %d: energies must be > 0 and finite", k, j);
        if (!(q.sigma_m2[i] >= 0.0) || !std::isfinite(q.sigma_m2[i]))
          return fail(SWARM_ERR_INVALID_ARG, "component %d channel %d: cross-sections must be >= 0 and finite", k, j);
        if (i > 0 && !(q.energy_eV[i] > q.energy_eV[i - 1]))
          return fail(SWARM_ERR_INVALID_ARG, "component %d channel %d: energies must increase strictly", k, j);
      }
      ++nc;
    }
  }
  if (std::fabs(fsum - 1.0) > 1e-9) return fail(SWARM_ERR_INVALID_ARG, "fractions sum to %.12g, not 1", fsum);
  if (nc > 4096) return fail(SWARM_ERR_INVALID_ARG, "too many channels (%d > 4096)", nc);
  return SWARM_OK;
}

hipError_t sync_desc_to_device(swarm* h) {
  return hipMemcpyAsync(h->d_desc, &h->desc, sizeof(InstanceDesc), hipMemcpyHostToDevice, h->stream);
}

// Tally tiles of a set of instances with known record counts.
void make_tiles(const std::vector<int64_t>& nrec, std::vector<TallyTile>& tiles, std::vector<int32_t>& base) {
  tiles.clear();
  base.assign(nrec.size(), 0);
  int32_t b = 0;
  for (size_t i = 0; i < nrec.size(); ++i) {
    base[i] = b;
    const int64_t nt = (nrec[i] + kTallyTile - 1) / kTallyTile;
    for (int64_t t = 0; t < nt; ++t) {
      TallyTile tt;
      tt.inst = static_cast<int32_t>(i);
      tt.tile = static_cast<int32_t>(t);
      tt.first = t * kTallyTile;
      tt.count = std::min<int64_t>(kTallyTile, nrec[i] - tt.first);
      tiles.push_back(tt);
    }
    b += static_cast<int32_t>(nt);
  }
}

}  // namespace

namespace swarm_impl {

hipError_t TallyPlan::prepare(const std::vector<int64_t>& nrec, hipStream_t s) {
  std::vector<TallyTile> tiles;
  std::vector<int32_t> base;
  make_tiles(nrec, tiles, base);
  n_inst = static_cast<int32_t>(nrec.size());
  n_tiles = static_cast<int32_t>(tiles.size());
  hipError_t e;
  if ((e = d_tiles.ensure(std::max<size_t>(1, tiles.size()) * sizeof(TallyTile))) != hipSuccess) return e;
  if ((e = d_base.ensure(base.size() * sizeof(int32_t))) != hipSuccess) return e;
  if ((e = d_nrec.ensure(nrec.size() * sizeof(int64_t))) != hipSuccess) return e;
  if ((e = d_part1.ensure(std::max<size_t>(1, tiles.size()) * kTally1 * sizeof(double))) != hipSuccess) return e;
  if ((e = d_part2.ensure(std::max<size_t>(1, tiles.size()) * kTally2 * sizeof(double))) != hipSuccess) return e;
  if ((e = d_tot.ensure(nrec.size() * (kTally1 + kTally2) * sizeof(double))) != hipSuccess) return e;
  if ((e = d_out.ensure(nrec.size() * sizeof(swarm_tallies_t))) != hipSuccess) return e;
  h_tiles = tiles;
  h_base = base;
  h_nrec = nrec;
  if (!tiles.empty() && (e = hipMemcpyAsync(d_tiles.p, h_tiles.data(), tiles.size() * sizeof(TallyTile),
                                            hipMemcpyHostToDevice, s)) != hipSuccess) return e;
  if ((e = hipMemcpyAsync(d_base.p, h_base.data(), base.size() * sizeof(int32_t), hipMemcpyHostToDevice, s)) != hipSuccess) return e;
  if ((e = hipMemcpyAsync(d_nrec.p, h_nrec.data(), nrec.size() * sizeof(int64_t), hipMemcpyHostToDevice, s)) != hipSuccess) return e;
  return hipSuccess;
}

hipError_t TallyPlan::launch(const InstanceDesc* d_descs, hipStream_t s) {
  if (n_tiles == 0) return hipSuccess;
  return launch_tallies(d_descs, static_cast<const TallyTile*>(d_tiles.p), n_tiles,
                        static_cast<const int32_t*>(d_base.p), static_cast<const int64_t*>(d_nrec.p), n_inst,
                        static_cast<double*>(d_part1.p), static_cast<double*>(d_part2.p),
                        static_cast<double*>(d_tot.p), static_cast<swarm_tallies_t*>(d_out.p), s);
}

// Team steps per collision: a step tests 2 g trials, each a hit with probability 1/t.
static double team_steps(double trials, int g) { return 1.0 / (1.0 - std::pow(1.0 - 1.0 / std::max(1.0, trials), 2.0 * g)); }

// Work per electron: a collision pass counts as about three trials; a team makes a step of 2 g
// trials at once, and its collision counts as about two and a half such steps.
double electron_work(double n_collisions, double trials, int team_lanes) {
  return n_collisions * (team_lanes <= 1 ? trials + 3.0 : team_steps(trials, team_lanes) + 2.5);
}

// The launch lasts about T, its work over its work-groups.  An instance whose electrons take w
// each can run floor(T / w) of them one after another in a lane, and starts with as many
// work-groups as that needs (all of its electrons at once where w is near T or above).  The
// longest electrons come first; instances that find no work-group left start when one is free.
// A work-group keeps its instance, with no wait between electrons, until the instance's
// electrons are all taken, and then helps another (next_instance).  Against
// a share in proportion to the work alone (ms): 16 adaptive argon swarms of 50,000 electrons,
// 2.4 a lane, 55.4 | 51.6, as it makes whole rounds; 40 uneven swarms of up to 10,000 electrons
// 33.2 | 29.5, as the longest electrons all start first; 20 argon fields x 60,000 93 | 94.
LaunchPlan plan_launch(const std::vector<int64_t>& n_e, const std::vector<double>& work, int64_t per_group, int64_t slots) {
  LaunchPlan p;
  const size_t n = n_e.size();
  std::vector<int64_t> most(n), given(n, 0);
  std::vector<int> order(n);
  int64_t groups = 0;
  double total = 0.0;
  for (size_t i = 0; i < n; ++i) {
    order[i] = static_cast<int>(i);
    most[i] = (n_e[i] + per_group - 1) / per_group;
    groups += most[i];
    total += static_cast<double>(most[i]) * work[i];
  }
  p.grid = static_cast<int>(std::max<int64_t>(1, std::min(groups, slots)));
  p.n_inst = static_cast<int32_t>(n);
  const double T = 0.9 * total / p.grid;     // (a margin: the work is an estimate)
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return work[a] > work[b]; });
  int64_t left = p.grid;
  for (int i : order) {
    const int64_t rounds = std::max<int64_t>(1, static_cast<int64_t>(std::min(T / work[i], 1e9)));
    given[i] = std::min(left, (most[i] + rounds - 1) / rounds);
    left -= given[i];
  }
  for (int i : order) {
    const int64_t more = std::min(left, most[i] - given[i]);
    given[i] += more;
    left -= more;
  }
  for (int i : order) p.lists.insert(p.lists.end(), given[i], static_cast<uint32_t>(i));
  for (double w : work) {
    const float f = std::max(1e-30f, static_cast<float>(w));
    uint32_t bits;
    std::memcpy(&bits, &f, sizeof(bits));
    p.lists.push_back(bits);
  }
  for (int64_t ne : n_e) p.lists.push_back(static_cast<uint32_t>(ne));
  return p;
}

hipError_t LaunchPlan::upload(void* base, hipStream_t s) const {
  return hipMemcpyAsync(static_cast<char*>(base) + counter_words() * 8, lists.data(), lists.size() * 4, hipMemcpyHostToDevice, s);
}
hipError_t LaunchPlan::clear(void* base, hipStream_t s) const {
  return launch_fill_u64(static_cast<uint64_t*>(base), 0ull, static_cast<int64_t>(counter_words()), s);
}
ClaimPlan LaunchPlan::view(void* base, int32_t chunk) const {
  const uint32_t* first = reinterpret_cast<const uint32_t*>(static_cast<char*>(base) + counter_words() * 8);
  const uint32_t* weight = first + grid;
  return {static_cast<unsigned long long*>(base), reinterpret_cast<const int32_t*>(first),
          reinterpret_cast<const float*>(weight), weight + n_inst, n_inst, chunk};
}
int32_t wave_chunk(const swarm_launch_opts& o) { return std::max(1, o.chunk / (o.block_size / 64)); }

// Default launch shape: work-groups of 256 (the autotuner's pick on MI355X for the argon-like
// sweep; 833 -> 789 ms per FP32 step against 128 with work items of that time).
int default_block() { return 256; }

swarm_launch_opts resolve_opts(const swarm_launch_opts* o) {
  swarm_launch_opts r{};
  const bool own = o && o->service_waves >= 0;      // (-1: the shape is left to the library)
  r.block_size = (own && o->block_size) ? o->block_size : default_block();
  // electrons the lanes of a work-group take at a time, one each: any number from a half to four
  // gave the same time (argon sweep 311 ms x 8000 collisions, FP64 252 to 255 ms x 2000)
  r.chunk = (own && o->chunk) ? o->chunk : r.block_size;
  r.use_graph = o ? o->use_graph : 0;
  r.block_size = std::max(64, std::min(1024, (r.block_size / 64) * 64));
  r.chunk = std::max(r.block_size, (r.chunk / r.block_size) * r.block_size);
  // (0 stays: every instance's own number, from the trials its collisions take)
  r.pending_trigger = own && o->pending_trigger ? std::max(1, std::min(64, o->pending_trigger)) : 0;
  r.service_waves = o ? std::max(0, std::min(r.block_size / 64 - 1, o->service_waves)) : 0;
  r.table_layout = (o && o->table_layout == 1) ? 1 : 0;
  r.park_lanes = (o && o->park_lanes) ? std::max(-1, std::min(64, o->park_lanes)) : kParkLanes;
  return r;
}

bool free_shape(const swarm_launch_opts* o) {
  return !o || o->service_waves < 0 ||
         (o->block_size == 0 && o->chunk == 0 && o->pending_trigger == 0 && o->service_waves == 0);
}

// A team of g lanes makes about one step per collision once 2 g exceeds the trials t that a
// collision takes, but it holds g lanes for it.  The launch is taken to last as long as its
// work at full occupancy plus its longest chain of collisions on a wave with a SIMD to itself;
// with the constants below (FP32, microseconds and lane instructions per collision, fitted to
// argon at 1 to 900 Td) that gives the runs of the table within 10 to 20%, and the g of the
// shortest one is taken.  Kernel ms, 800-1500 collisions, one lane at its best block and
// trigger | teams (g):
//   electrons                     25         1000         1e4         2e4        4e4        1e5
//   93:7 Ar:CO2 2.4 Td FP64   15.8|3.4(16) 19.5|3.5(16) 20.6|7.4(16) 22.2|10.2(8) 21.6|14.7(8) 29.3|30.2(2)
//   Ar:CO2 8 Td 0.5 T FP32     4.4|1.7(16)  5.7|1.7(16)  5.6|2.6(8)   6.0|3.1(8)   6.1|4.2(8)   7.1|7.7(2)
//   Ar:CO2 31 Td moving, FP32  3.4|2.0(8)   4.1|2.1(16)  4.1|2.7(8)   4.1|3.3(4)   4.3|4.1(4)   5.1|7.0(2)
//   argon 10 Td variable FP32  2.7|2.2(4)   3.8|2.4(8)   4.1|2.8(4)   4.4|3.1(4)   4.6|3.8(4)   5.3|5.8(2)
//   argon 100 Td FP64          3.2|2.1(8)   3.4|2.1(8)   3.4|2.3(4)   3.5|2.9(2)   3.6|4.1(2)   5.4|6.4(2)
//   argon 100 Td FP32          2.4|1.9(8)   2.7|1.9(8)   2.6|2.1(4)   2.8|2.4(4)   3.0|3.1(4)   3.9|4.7(2)
//   argon 900 Td FP32          1.9|1.8(4)   2.0|1.8(4)   2.0|2.0(4)   2.2|2.2(2)   2.4|2.6(2)   3.2|4.0(2)
//   Maxwell gas FP32           1.1|1.4(2)   1.1|1.4(2)   1.2|1.5(2)                1.6|1.9(2)   2.3|2.7(2)
// Few electrons whose collisions take many steps are spread over all SIMDs, fewer teams in a
// wave, so that a team waits less for the others (argon 1 Td, 1000 electrons: 2.6 against
// 3.3 ms); otherwise full waves are as fast.
TeamShape team_shape(const std::vector<int64_t>& n_e, const std::vector<double>& n_c, const std::vector<double>& trials) {
  const double simds = 4.0 * device_info().n_cu;
  const double slots_per_us = simds * 64 * 600.0;        // lane instructions, 2.4 GHz / 4
  TeamShape s;
  double best = 0.0, wide = 0.0, mean_t = 0.0, total_c = 0.0;
  for (size_t i = 0; i < n_e.size(); ++i) {
    const double c = static_cast<double>(n_e[i]) * n_c[i];
    mean_t += c * trials[i];
    total_c += c;
  }
  mean_t /= std::max(1.0, total_c);
  for (int g = 1; g <= 16; g *= 2) {
    double slots = 0.0, chain = 0.0, sum = 0.0;
    for (size_t i = 0; i < n_e.size(); ++i) {
      const double n = static_cast<double>(n_e[i]);
      double lanes, us;
      if (g == 1) {
        lanes = 100.0 * trials[i] + 60.0;
        us = 0.38 * trials[i] + 0.55;
      } else {
        const double steps = team_steps(trials[i], g);
        lanes = 260.0 * g * steps;
        us = 0.85 * steps + 0.35;
      }
      slots += n * n_c[i] * lanes;
      sum += n * n_c[i] * us;
      chain = std::max(chain, n_c[i] * us);
    }
    const double t = slots / slots_per_us + chain;
    if (g == 1 || t < best) {
      best = t;
      s.lanes = g;
      wide = chain > 0.0 ? sum / chain : 0.0;      // electrons that run at once, on average
    }
  }
  if (s.lanes == 1) return s;
  const int full = 64 / s.lanes;
  s.per_wave = mean_t < 6.0 ? full : static_cast<int>(std::min<double>(full, std::max(1.0, std::ceil(wide / simds))));
  s.block = wide <= simds * s.per_wave ? 64 : 256;
  return s;
}

}  // namespace swarm_impl

// =======================================================================================
// Single-instance API
// =======================================================================================
namespace swarm_impl {

// Validation, table build and constants of a new handle.  With bytes_only set, only the
// device bytes the handle's tables need are computed (nothing is allocated or launched).
static swarm_status build_swarm(swarm* h, const swarm_component* comps, int32_t n_comps,
                                const swarm_params* params, size_t* bytes_only) {
  swarm_status st = validate(comps, n_comps, params);
  if (st != SWARM_OK) return st;
  h->params = *params;
  // Flatten the raw tables (argument marshalling only).
  std::vector<double> e_all, s_all, thr, mass, frac, ratio;
  std::vector<int32_t> off, npt, kind, comp, scat;
  for (int k = 0; k < n_comps; ++k) {
    mass.push_back(comps[k].mass_amu);
    frac.push_back(comps[k].fraction);
    scat.push_back(comps[k].scattering);
    ratio.push_back(comps[k].scattering == SWARM_SCATTER_CONSTANT_XI ? comps[k].mt_over_el : 1.0);
    for (int j = 0; j < comps[k].n_channels; ++j) {
      const swarm_channel& q = comps[k].channels[j];
      off.push_back(static_cast<int32_t>(e_all.size()));
      npt.push_back(q.n_points);
      kind.push_back(q.kind);
      comp.push_back(k);
      thr.push_back(q.threshold_eV);
      e_all.insert(e_all.end(), q.energy_eV, q.energy_eV + q.n_points);
      s_all.insert(s_all.end(), q.sigma_m2, q.sigma_m2 + q.n_points);
      h->kinds.push_back(q.kind);
    }
  }
  const int nc = static_cast<int>(off.size());
  const int P = params->grid_points_per_octave ? params->grid_points_per_octave : 64;
  int emin = params->grid_min_exp2, emax = params->grid_max_exp2;
  if (emin == 0 && emax == 0) { emin = -14; emax = 12; }
  int p_log2 = 0;
  while ((1 << p_log2) < P) ++p_log2;
  const int G = (emax - emin) * P + 1;
  InstanceDesc& d = h->desc;
  std::memset(&d, 0, sizeof(d));
  d.G = G; d.nc = nc; d.p_log2 = p_log2; d.emin = emin; d.emax = emax; d.n_raw_channels = nc;
  d.precision = params->precision; d.secondaries = params->secondaries;
  d.E = params->E_V_per_m; d.B = params->B_T; d.B_angle = params->B_angle_rad; d.N = params->N_per_m3;
  d.eps0 = params->init_energy_eV; d.user_majorant = params->user_majorant;
  d.T_K = params->T_K; d.thermal_targets = params->thermal_targets; d.relativistic = params->relativistic;
  d.trial_strategy = params->trial_strategy;
  d.trial_zeta = params->trial_zeta > 0.0 ? params->trial_zeta : 0.25;
  d.trial_grace = static_cast<uint32_t>(params->trial_grace > 0 ? params->trial_grace : 5000);
  d.trial_bins = params->trial_bins > 0 ? params->trial_bins : 10;
  std::vector<int32_t> entry_bin, bin_first;
  if (params->trial_strategy == SWARM_TRIAL_BINNED) decade_bins(P, emin, G, d.trial_bins, entry_bin, bin_first);
  d.balance_node = static_cast<uint32_t>(G - 1);
  d.n_bins = entry_bin.empty() ? 0 : static_cast<int32_t>(bin_first.size()) - 1;
  h->has_b = params->B_T > 0.0;
  // one arena for the raw inputs and the tables
  auto al = [](size_t n) { return (n + 255) & ~size_t(255); };
  const size_t b_e = al(e_all.size() * 8), b_s = b_e, b_i = al(nc * 4), b_cd = al(nc * 8), b_k = al(n_comps * 8);
  const size_t b_nodes = al(static_cast<size_t>(G) * 8);
  const size_t b_cm = al(static_cast<size_t>(G) * nc * 8);
  const size_t b_nu64 = al(static_cast<size_t>(G) * 16), b_nu32 = al(static_cast<size_t>(G) * 8);
  // running sums, node major, padded with a row in front (below the grid), with spare pairs
  // after the last row (the channel search reads a whole row of up to 8 pairs at once)
  const size_t b_c64 = al((static_cast<size_t>(G + 1) * nc + 8) * 16), b_c32 = al((static_cast<size_t>(G + 1) * nc + 8) * 8);
  const size_t b_ch = al(nc * sizeof(ChannelDev)), b_th = al(nc * sizeof(ThermalChannel));
  const size_t b_eb = al(entry_bin.size() * 4), b_bf = al(bin_first.size() * 4);
  const size_t b_bn = al(static_cast<size_t>(d.n_bins) * 8), b_bn32 = al(static_cast<size_t>(d.n_bins) * 4);
  std::vector<double> logtab(kUnitLogStride * kUnitLogEntries);
  unit_log_table(logtab.data());
  const size_t b_lt = al(logtab.size() * 8);
  const size_t total = b_e + b_s + 4 * b_i + b_cd + 4 * b_k + b_nodes + b_cm + b_nu64 + b_nu32 + b_c64 + b_c32 + b_ch +
                       b_th + b_eb + b_bf + b_bn + b_bn32 + b_lt + al(sizeof(InstanceDesc)) + al(sizeof(RunCounters));
  if (bytes_only) {
    *bytes_only = total;
    return SWARM_OK;
  }
  if (params->stream) {
    h->stream = static_cast<hipStream_t>(params->stream);
    h->own_stream = false;
  } else {
    hipError_t es = hipStreamCreateWithFlags(&h->stream, hipStreamNonBlocking);
    if (es != hipSuccess) return hip_fail(es, "hipStreamCreate");
    h->own_stream = true;
  }
  hipError_t e = h->arena.ensure(total);
  if (e != hipSuccess) return hip_fail(e, "allocating instance tables");
  char* base = static_cast<char*>(h->arena.p);
  size_t o = 0;
  auto take = [&](size_t n) { char* r = base + o; o += n; return r; };
  double* d_e = reinterpret_cast<double*>(take(b_e));
  double* d_s = reinterpret_cast<double*>(take(b_s));
  int32_t* d_off = reinterpret_cast<int32_t*>(take(b_i));
  int32_t* d_n = reinterpret_cast<int32_t*>(take(b_i));
  int32_t* d_kind = reinterpret_cast<int32_t*>(take(b_i));
  int32_t* d_comp = reinterpret_cast<int32_t*>(take(b_i));
  double* d_thr = reinterpret_cast<double*>(take(b_cd));
  double* d_mass = reinterpret_cast<double*>(take(b_k));
  double* d_frac = reinterpret_cast<double*>(take(b_k));
  int32_t* d_scat = reinterpret_cast<int32_t*>(take(b_k));
  double* d_ratio = reinterpret_cast<double*>(take(b_k));
  d.nodes = reinterpret_cast<double*>(take(b_nodes));
  d.cum_cm = reinterpret_cast<double*>(take(b_cm));
  d.nu64 = reinterpret_cast<double2*>(take(b_nu64));
  d.nu32 = reinterpret_cast<float2*>(take(b_nu32));
  d.cum64 = reinterpret_cast<double2*>(take(b_c64));
  d.cum32 = reinterpret_cast<float2*>(take(b_c32));
  d.chan = reinterpret_cast<ChannelDev*>(take(b_ch));
  d.chan_th = reinterpret_cast<ThermalChannel*>(take(b_th));
  int32_t* d_entry_bin = reinterpret_cast<int32_t*>(take(b_eb));
  int32_t* d_bin_first = reinterpret_cast<int32_t*>(take(b_bf));
  d.bin_of = d_entry_bin;
  d.bin_first = d_bin_first;
  d.bin_nup64 = reinterpret_cast<double*>(take(b_bn));
  d.bin_nup32 = reinterpret_cast<float*>(take(b_bn32));
  double* d_logtab = reinterpret_cast<double*>(take(b_lt));
  d.logtab = d_logtab;
  h->d_desc = reinterpret_cast<InstanceDesc*>(take(al(sizeof(InstanceDesc))));
  d.ctr = reinterpret_cast<RunCounters*>(take(al(sizeof(RunCounters))));
  d.raw_e = d_e; d.raw_s = d_s; d.raw_off = d_off; d.raw_n = d_n; d.raw_kind = d_kind;
  d.raw_comp = d_comp; d.raw_thr = d_thr; d.comp_mass_amu = d_mass; d.comp_frac = d_frac;
  d.comp_scat = d_scat; d.comp_ratio = d_ratio;
  hipStream_t s = h->stream;
#define CP(dst, v) if ((e = hipMemcpyAsync(dst, v.data(), v.size() * sizeof(v[0]), hipMemcpyHostToDevice, s)) != hipSuccess) return hip_fail(e, "copying tables");
  CP(d_e, e_all) CP(d_s, s_all) CP(d_off, off) CP(d_n, npt) CP(d_kind, kind) CP(d_comp, comp)
  CP(d_thr, thr) CP(d_mass, mass) CP(d_frac, frac) CP(d_scat, scat) CP(d_ratio, ratio)
  if (!entry_bin.empty()) { CP(d_entry_bin, entry_bin) CP(d_bin_first, bin_first) }
  CP(d_logtab, logtab)
#undef CP
  if ((e = launch_fill_u64(reinterpret_cast<uint64_t*>(d.ctr), 0, sizeof(RunCounters) / 8, s)) != hipSuccess)
    return hip_fail(e, "clearing counters");
  if ((e = sync_desc_to_device(h)) != hipSuccess) return hip_fail(e, "copying descriptor");
  if ((e = launch_build(h->d_desc, d, s)) != hipSuccess) return hip_fail(e, "table build launch");
  if ((e = hipMemcpyAsync(&h->desc, h->d_desc, sizeof(InstanceDesc), hipMemcpyDeviceToHost, s)) != hipSuccess)
    return hip_fail(e, "reading descriptor");
  if ((e = hipStreamSynchronize(s)) != hipSuccess) return hip_fail(e, "table build");
  if (h->desc.built_ok == -1)
    return fail(SWARM_ERR_INVALID_ARG, "the total collision frequency vanishes on part of the energy grid");
  if (h->desc.built_ok == -2)
    return fail(SWARM_ERR_INVALID_ARG, "user trial frequency %.6g is below the maximum collision frequency %.6g",
                params->user_majorant, h->desc.numax);
  if (h->desc.built_ok != 1) return fail(SWARM_ERR_DEVICE, "table build did not complete");
  for (int i = 0; i < 3; ++i)
    if ((e = hipEventCreate(&h->ev[i])) != hipSuccess) return hip_fail(e, "hipEventCreate");
  // (Single runs of a swarm take the same default as batches.  Work-groups of 128 were better
  // while draining waves waited for their last lane; since they do not, 256 with the trigger of
  // the instance is: 1e5 electrons x 2000 argon collisions at 100 Td, FP64 13.4 -> 9.7 ms, FP32
  // 6.0 -> 4.9 ms, at 1 Td 64.5 -> 62.9 and 28.7 -> 28.1 ms.)
  h->opts = resolve_opts(nullptr);
  return SWARM_OK;
}

swarm_status create_swarm(const swarm_component* comps, int32_t n_comps, const swarm_params* params,
                          Arena* mem, swarm_t* out) {
  if (!out) return fail(SWARM_ERR_INVALID_ARG, "out is NULL");
  *out = nullptr;
  auto h = std::make_unique<swarm>();
  if (mem) h->bind_arena(mem);
  const swarm_status st = build_swarm(h.get(), comps, n_comps, params, nullptr);
  if (st != SWARM_OK) {
    const std::string msg = g_last_error;
    swarm_destroy(h.release());
    g_last_error = msg;
    return st;
  }
  *out = h.release();
  return SWARM_OK;
}

size_t create_bytes(const swarm_component* comps, int32_t n_comps, const swarm_params* params) {
  swarm h;
  size_t bytes = 0;
  if (build_swarm(&h, comps, n_comps, params, &bytes) != SWARM_OK) return 0;
  return bytes;
}

}  // namespace swarm_impl

extern "C" {

const char* swarm_strerror(swarm_status s) {
  switch (s) {
    case SWARM_OK: return "ok";
    case SWARM_ERR_INVALID_ARG: return "invalid argument";
    case SWARM_ERR_OUT_OF_MEMORY: return "out of memory";
    case SWARM_ERR_CAPACITY: return "capacity exceeded";
    case SWARM_ERR_DEVICE: return "device error";
    case SWARM_ERR_STATE: return "invalid state";
    case SWARM_PENDING: return "pending";
  }
  return "unknown status";
}

const char* swarm_last_error(void) { return g_last_error.c_str(); }

swarm_status swarm_create(const swarm_component* comps, int32_t n_comps, const swarm_params* params,
                          swarm_t* out) {
  return create_swarm(comps, n_comps, params, nullptr, out);
}

swarm_status swarm_create_in_arena(const swarm_component* comps, int32_t n_comps, const swarm_params* params,
                                   void* arena, int64_t arena_bytes, swarm_t* out) {
  if (!out) return fail(SWARM_ERR_INVALID_ARG, "out is NULL");
  *out = nullptr;
  if (!arena || arena_bytes <= 0) return fail(SWARM_ERR_INVALID_ARG, "arena must be a device pointer with bytes > 0");
  auto mem = std::make_unique<Arena>(arena, static_cast<size_t>(arena_bytes));
  swarm_t h = nullptr;
  const swarm_status st = create_swarm(comps, n_comps, params, mem.get(), &h);
  if (st != SWARM_OK) return st;
  h->own_mem = std::move(mem);
  *out = h;
  return SWARM_OK;
}

swarm_status swarm_arena_bytes(const swarm_component* comps, int32_t n_comps, const swarm_params* params,
                               int64_t n_electrons, int64_t* bytes) {
  if (!bytes) return fail(SWARM_ERR_INVALID_ARG, "bytes is NULL");
  *bytes = 0;
  if (n_electrons < 1) return fail(SWARM_ERR_INVALID_ARG, "n_electrons must be >= 1");
  const size_t tables = create_bytes(comps, n_comps, params);
  if (tables == 0) return SWARM_ERR_INVALID_ARG;     // validation failed; the message is set
  auto blk = [](size_t n) { return (n + 2 * 256 - 1) & ~static_cast<size_t>(255); };   // block + alignment
  const bool real = params->secondaries == SWARM_REAL;
  const int64_t capacity = real ? (params->capacity ? params->capacity : 64 * n_electrons) : n_electrons;
  size_t run = blk(static_cast<size_t>(capacity) * sizeof(swarm_record)) + tally_bytes(capacity);
  if (real && capacity > n_electrons) run += blk(static_cast<size_t>(capacity - n_electrons) * sizeof(ChildState));
  // real mode: the two buffers of parked electrons, for the most lanes a device can hold
  if (real) run += blk(2 * static_cast<size_t>(parked_capacity(static_cast<int64_t>(device_info().n_cu) * 2048, 64)) * sizeof(ParkedState));
  *bytes = static_cast<int64_t>(blk(tables) + run);
  return SWARM_OK;
}

void swarm_destroy(swarm_t h) {
  if (!h) return;
  if (h->worker.joinable()) h->worker.join();
  if (h->stream) (void)hipStreamSynchronize(h->stream);
  for (int i = 0; i < 3; ++i)
    if (h->ev[i]) (void)hipEventDestroy(h->ev[i]);
  if (h->own_stream && h->stream) (void)hipStreamDestroy(h->stream);
  delete h;
}

swarm_status swarm_set_trace(swarm_t h, const uint64_t* ids, int32_t n_ids, int32_t max_events) {
  if (!h) return fail(SWARM_ERR_INVALID_ARG, "handle is NULL");
  if (h->in_flight) return busy();
  if (n_ids < 0 || n_ids > kMaxTraceIds) return fail(SWARM_ERR_INVALID_ARG, "n_ids must be in [0, %d]", kMaxTraceIds);
  if (n_ids > 0 && (!ids || max_events <= 0 || max_events > 4096))
    return fail(SWARM_ERR_INVALID_ARG, "max_events must be in [1, 4096]");
  h->n_trace = n_ids;
  h->max_events = n_ids ? max_events : 0;
  if (n_ids == 0) return SWARM_OK;
  hipError_t e;
  if ((e = h->trace_ids.ensure(n_ids * sizeof(uint64_t))) != hipSuccess) return hip_fail(e, "trace ids");
  if ((e = h->trace_out.ensure(static_cast<size_t>(n_ids) * max_events * sizeof(swarm_event))) != hipSuccess)
    return hip_fail(e, "trace buffer");
  if ((e = h->trace_count.ensure(n_ids * sizeof(int32_t))) != hipSuccess) return hip_fail(e, "trace counts");
  if ((e = hipMemcpyAsync(h->trace_ids.p, ids, n_ids * sizeof(uint64_t), hipMemcpyHostToDevice, h->stream)) != hipSuccess)
    return hip_fail(e, "trace ids");
  if ((e = hipStreamSynchronize(h->stream)) != hipSuccess) return hip_fail(e, "trace ids");
  return SWARM_OK;
}

swarm_status swarm_set_launch_opts(swarm_t h, const swarm_launch_opts* opts) {
  if (!h) return fail(SWARM_ERR_INVALID_ARG, "NULL handle");
  if (h->in_flight) return busy();
  h->opts = resolve_opts(opts);
  h->free_shape = free_shape(opts);
  return SWARM_OK;
}

}  // extern "C"

namespace {

// A run up to the point where everything is on the stream: records, counters, the swarm
// kernel (dummy mode: one launch; real mode: the generations, which need the host between
// launches and therefore wait for each), then the tally reductions.  Nothing waits for the
// dummy-mode work, so swarm_run_async returns while it runs.  A capacity overflow is kept
// in run_status: its tallies are still reduced.
swarm_status run_start(swarm_t h, int64_t n_electrons, int64_t n_collisions, uint64_t seed) {
  if (n_electrons < 1) return fail(SWARM_ERR_INVALID_ARG, "n_electrons must be >= 1");
  if (n_collisions < 1 || n_collisions > 0xffffffffLL)
    return fail(SWARM_ERR_INVALID_ARG, "n_collisions must be in [1, 2^32-1]");
  h->run_status = SWARM_OK;
  h->run_error.clear();
  h->noalloc_records = false;
  const bool real = h->desc.secondaries == SWARM_REAL;
  int64_t capacity = n_electrons;
  if (real) {
    capacity = h->params.capacity ? h->params.capacity : 64 * n_electrons;
    if (capacity < n_electrons) return fail(SWARM_ERR_INVALID_ARG, "capacity below n_electrons");
  }
  hipStream_t s = h->stream;
  hipError_t e;
  h->have_run = false;
  if ((e = h->records.ensure(static_cast<size_t>(capacity) * sizeof(swarm_record))) != hipSuccess)
    return hip_fail(e, "allocating records");
  InstanceDesc& d = h->desc;
  d.n_electrons = n_electrons;
  d.n_collisions = static_cast<uint32_t>(n_collisions);
  d.quantum = 0;
  d.seed = seed;
  d.capacity = capacity;
  d.records = static_cast<swarm_record*>(h->records.p);
  d.saved = nullptr;
  d.children = nullptr;
  const int64_t child_cap = capacity - n_electrons;
  if (real && child_cap > 0) {
    if ((e = h->children.ensure(static_cast<size_t>(child_cap) * sizeof(ChildState))) != hipSuccess)
      return hip_fail(e, "allocating secondary queue");
    d.children = static_cast<ChildState*>(h->children.p);
  }
  if (real && (e = launch_mark_empty(d.records, capacity, s)) != hipSuccess) return hip_fail(e, "clearing records");
  const bool trace = h->n_trace > 0;
  d.trace_ids = trace ? static_cast<const uint64_t*>(h->trace_ids.p) : nullptr;
  d.n_trace = h->n_trace;
  d.max_events = h->max_events;
  d.trace_out = trace ? static_cast<swarm_event*>(h->trace_out.p) : nullptr;
  d.trace_count = trace ? static_cast<int32_t*>(h->trace_count.p) : nullptr;
  if (trace && (e = launch_fill_u32(reinterpret_cast<uint32_t*>(d.trace_count), 0u, h->n_trace, s)) != hipSuccess)
    return hip_fail(e, "clearing trace counts");
  // counters: all zero
  if ((e = launch_fill_u64(reinterpret_cast<uint64_t*>(d.ctr), 0ull, sizeof(RunCounters) / sizeof(uint64_t), s)) != hipSuccess)
    return hip_fail(e, "counters");
  if ((e = sync_desc_to_device(h)) != hipSuccess) return hip_fail(e, "descriptor");
  const swarm_launch_opts& o = h->opts;
  const int svc = trace || real ? 0 : o.service_waves;
  const LdsLayout ll = lds_layout(d.precision, d.G, d.nc, svc, o.table_layout);
  if (static_cast<int64_t>(ll.bytes) > device_info().lds_per_block)
    return fail(SWARM_ERR_INVALID_ARG, "the tables need %zu bytes of LDS per work-group, the device has %lld",
                ll.bytes, static_cast<long long>(device_info().lds_per_block));
  const size_t lds = ll.bytes;
  const int ch_off = ll.ch_off;
  DeviceInfo& dev = device_info();
  const int ext = d.thermal_targets || d.relativistic ? 2 : d.trial_strategy != SWARM_TRIAL_CONSTANT ? 1 : 0;
  const int per_cu = swarm_kernel_max_blocks_per_cu(d.precision, h->has_b, trace, real, ext, svc, o.block_size, lds);
  const bool may_team = h->free_shape && !trace;
  auto team_grid = [&](const TeamShape& t, int64_t groups) {
    const int64_t resident = static_cast<int64_t>(dev.n_cu) *
                             swarm_kernel_max_blocks_per_cu(d.precision, h->has_b, false, real, ext, 0, t.block, lds, true);
    return static_cast<int>(std::max<int64_t>(1, std::min(groups, resident)));
  };
  if ((e = hipEventRecord(h->ev[0], s)) != hipSuccess) return hip_fail(e, "event");
  if (!real) {
    const TeamShape team = may_team ? team_shape({n_electrons}, {static_cast<double>(n_collisions)}, {d.trials}) : TeamShape{};
    const int64_t per_group = team.lanes > 1 ? team.per_group() : o.block_size;
    const int64_t groups = (n_electrons + per_group - 1) / per_group;
    const int grid = team.lanes > 1 ? team_grid(team, groups)
                                    : static_cast<int>(std::min<int64_t>(groups, static_cast<int64_t>(dev.n_cu) * per_cu));
    const ClaimPlan plan = {reinterpret_cast<unsigned long long*>(&d.ctr->gen_next), nullptr, nullptr, nullptr, 1, wave_chunk(o)};
    if ((e = launch_swarm_dummy(h->d_desc, plan, d.precision, h->has_b, trace, ext, svc, o.block_size, grid, o.pending_trigger,
                                lds, ch_off, ll.pool_off, ll.cum_off, s, team)) != hipSuccess)
      return hip_fail(e, "swarm kernel launch");
    h->team_lanes = team.lanes;
    h->n_launches = 1;
    h->n_parked = 0;
  }
  RunCounters hc{};
  if (real) {
    // One launch per generation: the primaries, then the secondaries each generation
    // appended to the queue (slots [first, first + count)), until a generation creates none.
    // Every generation starts at least one collision later in its lineage budget than the
    // one before, so there are at most n_collisions + 1.  After an overflow the next launch
    // records the queued secondaries unstarted (flag 8) and creates none.
    //
    // Small runs, and the ends of all, go in slices of the lineage budget (SlicePlan).  Ar:CO2
    // mixture, ms with whole generations and with slices of 64, 128, 256 collisions from the start,
    // at 1 T: 500 primaries x 1500, FP32 18.0, 8.4, 10.0, 12.0, FP64 31.5, 13.7, 16.4, 20.6; 5000 x
    // 1500, FP32 23.0, 16.2, 14.9, 17.4, FP64 38.9, 23.7, 25.0, 27.6.  With up to 100,000 electrons
    // sliced from the start and none, or again 100,000, at the end: 100,000 x 2000 FP32 69.7 and
    // 64.8, 50,000 x 1000 at B = 0 16.2 and 14.8.  With up to 30,000, 50,000 and 100,000 at the start
    // and 100,000 at the end: the same runs 65.4, 65.4, 64.8 and 14.4, 15.0, 14.8, FP64 20,000 x
    // 1000 17.8, 17.2, 20.1 and 60,000 x 600 8.7, 8.6, 11.8; with 200,000 at the end 66.0, 15.3, 20.1
    // and 11.8, with 50,000 67.5, 14.4, 18.9 and 9.0.
    // Where little is ionised, FP32 with whole generations, slices of 64 or 128 throughout and
    // growing ones: the mixture at 5 Td, 20,000 x 3000, 11.5, 21.2, 13.4, argon at 10 Td, 5000 x
    // 5000, 10.1, 18.0, 12.3, at 50 Td, 1000 x 10,000 (11,600 electrons in the end), 102, 38.7, 38.4,
    // the Maxwell gas, 30,000 x 3000, 2.8, 12.1 and never sliced.
    //
    // Beyond that, a launch that has created secondaries for at least an eighth of the device's
    // lanes lets its last few running electrons park (1e6 primaries: FP32 399 -> 372 ms, FP64
    // 1004 -> 966 ms; waves of at most 16 running lanes parking after half a device of
    // secondaries: 379 and 988 ms; 48 lanes after a sixteenth: 384 and 960 ms).
    //
    // No more than four waves per SIMD.  The collisions of a magnetised mixture wait on L2, and the
    // channel rows of more waves crowd it (100,000 primaries 73.3 ms with five, 70.4 with four, 72.0
    // with three; 1e6 primaries x 1000 76.6 and 72.4 with five and four).  Argon's five channels
    // do not, but its generations of some rounds end earlier too on fewer lanes (FP32, five and four:
    // 300,000 x 1000 at 100 Td 28.0 and 25.9, x 1500 at 30 Td 15.5 and 14.6, 1e6 x 100 at 100 Td 6.8
    // and 6.3); where many primaries ionise little it would gain from five (1e6 x 300 at 30 Td 8.9
    // and 9.7, 1e6 x 1000 at 10 Td 24.5 and 25.7).
    const int groups_per_cu = std::max(1, std::min(per_cu, 16 * 64 / o.block_size));
    const int64_t lanes = static_cast<int64_t>(dev.n_cu) * groups_per_cu * o.block_size;
    const int park_lanes = std::max(0, o.park_lanes);   // -1: never
    // (where memory cannot hold the parked electrons of slices, those of a launch's end)
    const int64_t end_cap = parked_capacity(lanes, park_lanes);
    const int64_t slice_lanes = static_cast<int64_t>(dev.n_cu) * 4 * 4 * 64;
    int64_t park_cap = park_lanes == 0 ? end_cap : std::max(end_cap, std::min(capacity, slice_lanes / 8 * 3));
    e = h->parked.ensure(2 * static_cast<size_t>(park_cap) * sizeof(ParkedState));
    if (e == hipErrorOutOfMemory && park_cap > end_cap) {
      (void)hipGetLastError();
      park_cap = end_cap;
      e = h->parked.ensure(2 * static_cast<size_t>(park_cap) * sizeof(ParkedState));
    }
    if (e != hipSuccess) return hip_fail(e, "allocating parked electrons");
    ParkedState* park_in = static_cast<ParkedState*>(h->parked.p);
    ParkedState* park_out = park_in + park_cap;
    const bool ionises = std::find(h->kinds.begin(), h->kinds.end(), SWARM_IONIZATION) != h->kinds.end();
    SlicePlan slices = {n_collisions, slice_lanes, park_cap, ionises && park_lanes > 0};
    int64_t first = -1, count = n_electrons, queued = 0, n_parked = 0;
    h->n_launches = 0;
    h->n_parked = 0;
    h->team_lanes = 1;
    for (;;) {
      if ((e = launch_next_generation(d.ctr, s)) != hipSuccess) return hip_fail(e, "generation counters");
      const int64_t electrons = n_parked + count;
      const int64_t want = (electrons + o.block_size - 1) / o.block_size;
      const TeamShape team = may_team ? team_shape({electrons}, {static_cast<double>(n_collisions)}, {d.trials}) : TeamShape{};
      // (the triggers of k_build_constants are for launches whose draining waves do not park)
      constexpr int kRealTrigger = 32;
      const int grid = team.lanes > 1
          ? team_grid(team, (electrons + team.per_group() - 1) / team.per_group())
          : static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(want, static_cast<int64_t>(dev.n_cu) * groups_per_cu)));
      const int64_t limit = slices.limit(electrons);
      const uint32_t slice = slices.sliced ? static_cast<uint32_t>(std::min(slices.length, n_collisions)) : 0u;
      const int64_t park_min = hc.dropped != 0 || park_lanes == 0 ? 0 : std::max<int64_t>(1, lanes / 8);
      if ((e = launch_swarm_real(h->d_desc, d.precision, h->has_b, trace, ext, o.block_size, grid,
                                 o.pending_trigger ? o.pending_trigger : kRealTrigger, lds,
                                 ch_off, ll.cum_off, first, count, hc.dropped != 0 ? 1 : 0, park_in, n_parked, park_out,
                                 park_min, park_lanes, queued, static_cast<uint32_t>(limit), slice, park_cap, s, team)) != hipSuccess)
        return hip_fail(e, "swarm kernel launch");
      h->n_launches += 1;
      h->team_lanes = std::max(h->team_lanes, team.lanes);
      if ((e = hipMemcpyAsync(&hc, d.ctr, sizeof(hc), hipMemcpyDeviceToHost, s)) != hipSuccess) return hip_fail(e, "counters");
      if ((e = hipStreamSynchronize(s)) != hipSuccess) return hip_fail(e, "swarm kernel");
      const int64_t tail = std::min<int64_t>(static_cast<int64_t>(hc.child_tail), child_cap);
      if (tail == queued && hc.parked == 0) break;   // no secondary created, none parked
      first = queued;
      count = tail - queued;
      queued = tail;
      n_parked = std::min<int64_t>(static_cast<int64_t>(hc.parked), park_cap);
      slices.launched(electrons, count, limit, static_cast<int64_t>(hc.k_min));
      h->n_parked += n_parked;
      std::swap(park_in, park_out);
    }
  }
  if ((e = hipEventRecord(h->ev[1], s)) != hipSuccess) return hip_fail(e, "event");
  if (real) {
    if ((e = hipMemcpyAsync(&hc, d.ctr, sizeof(hc), hipMemcpyDeviceToHost, s)) != hipSuccess) return hip_fail(e, "counters");
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return hip_fail(e, "swarm kernel");
  }
  h->n_records = n_electrons + (real ? std::min<int64_t>(static_cast<int64_t>(hc.child_tail), child_cap) : 0);
  if ((e = h->tally.prepare({h->n_records}, s)) != hipSuccess) return hip_fail(e, "tally plan");
  if ((e = h->tally.launch(h->d_desc, s)) != hipSuccess) return hip_fail(e, "tally launch");
  if ((e = hipEventRecord(h->ev[2], s)) != hipSuccess) return hip_fail(e, "event");
  h->traced = trace;
  if (hc.dropped) {
    h->run_status = fail(SWARM_ERR_CAPACITY, "%llu secondaries did not fit the capacity of %lld electrons",
                         static_cast<unsigned long long>(hc.dropped), static_cast<long long>(capacity));
    h->run_error = g_last_error;
  }
  return SWARM_OK;
}

// Wait for the enqueued run, read its tallies and timings back.
swarm_status run_finish(swarm_t h) {
  hipError_t e;
  if ((e = hipEventSynchronize(h->ev[2])) != hipSuccess) return hip_fail(e, "swarm run");
  if ((e = hipMemcpyAsync(&h->tallies, h->tally.d_out.p, sizeof(swarm_tallies_t), hipMemcpyDeviceToHost,
                          h->stream)) != hipSuccess ||
      (e = hipStreamSynchronize(h->stream)) != hipSuccess)
    return hip_fail(e, "tallies");
  float ms = 0.f;
  (void)hipEventElapsedTime(&ms, h->ev[0], h->ev[1]);
  h->kernel_ms = ms;
  (void)hipEventElapsedTime(&ms, h->ev[0], h->ev[2]);
  h->total_ms = ms;
  h->have_run = true;
  if (h->run_status != SWARM_OK) g_last_error = h->run_error;
  return h->run_status;
}

}  // namespace

extern "C" {

swarm_status swarm_run(swarm_t h, int64_t n_electrons, int64_t n_collisions, uint64_t seed) {
  if (!h) return fail(SWARM_ERR_INVALID_ARG, "handle is NULL");
  if (h->in_flight) return busy();
  const swarm_status st = run_start(h, n_electrons, n_collisions, seed);
  if (st != SWARM_OK) return st;
  return run_finish(h);
}

swarm_status swarm_run_async(swarm_t h, int64_t n_electrons, int64_t n_collisions, uint64_t seed) {
  if (!h) return fail(SWARM_ERR_INVALID_ARG, "handle is NULL");
  if (h->in_flight) return busy();
  h->have_run = false;
  if (h->desc.secondaries == SWARM_REAL) {
    // the generations need the host between launches: they run on a worker thread
    if (n_electrons < 1 || n_collisions < 1 || n_collisions > 0xffffffffLL)
      return fail(SWARM_ERR_INVALID_ARG, "n_electrons must be >= 1 and n_collisions in [1, 2^32-1]");
    h->in_flight = 2;
    h->worker = std::thread([h, n_electrons, n_collisions, seed] {
      swarm_status st = run_start(h, n_electrons, n_collisions, seed);
      if (st == SWARM_OK) st = run_finish(h);
      h->async_status = st;
      h->async_error = st != SWARM_OK ? g_last_error : std::string();
    });
    return SWARM_OK;
  }
  const swarm_status st = run_start(h, n_electrons, n_collisions, seed);
  if (st != SWARM_OK) return st;
  h->in_flight = 1;
  return SWARM_OK;
}

swarm_status swarm_wait(swarm_t h) {
  if (!h) return fail(SWARM_ERR_INVALID_ARG, "handle is NULL");
  if (h->in_flight == 0) return fail(SWARM_ERR_STATE, "no run in flight");
  if (h->in_flight == 2) {
    h->worker.join();
    h->in_flight = 0;
    if (h->async_status != SWARM_OK) g_last_error = h->async_error;
    return h->async_status;
  }
  h->in_flight = 0;
  return run_finish(h);
}

swarm_status swarm_tallies(swarm_t h, swarm_tallies_t* out) {
  if (!h || !out) return fail(SWARM_ERR_INVALID_ARG, "NULL argument");
  if (h->in_flight) return busy();
  if (!h->have_run) return fail(SWARM_ERR_STATE, "no completed run");
  *out = h->tallies;
  return SWARM_OK;
}

swarm_status swarm_records(swarm_t h, swarm_record* out, int64_t max_records, int64_t* n_out) {
  if (!h || !n_out) return fail(SWARM_ERR_INVALID_ARG, "NULL argument");
  if (h->in_flight) return busy();
  if (h->noalloc_records) return fail(SWARM_ERR_STATE, "the last run wrote its records to caller memory");
  if (!h->have_run) return fail(SWARM_ERR_STATE, "no completed run");
  // A complete run has a record in every slot: counted without a copy, and copied straight to the
  // caller (through a vector and twice, to count first, the 100,000 records of an FP64 point
  // took 2.6-6.6 ms beside 10 ms of simulation; straight, 1.2-3.0).
  if (h->run_status == SWARM_OK) {
    *n_out = h->n_records;
    const int64_t n = std::min(h->n_records, max_records);
    if (!out || n <= 0) return SWARM_OK;
    hipError_t e = hipMemcpyAsync(out, h->desc.records, static_cast<size_t>(n) * sizeof(swarm_record),
                                  hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    return e == hipSuccess ? SWARM_OK : hip_fail(e, "copying records");
  }
  // Slots of secondaries that a run stopped early never simulated are empty (id all ones)
  // and are left out: *n_out counts the electrons that have a record.
  std::vector<swarm_record> all(static_cast<size_t>(h->n_records));
  if (h->n_records > 0) {
    hipError_t e = hipMemcpyAsync(all.data(), h->desc.records, all.size() * sizeof(swarm_record),
                                  hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) return hip_fail(e, "copying records");
  }
  int64_t n = 0;
  for (const swarm_record& r : all) {
    if (r.id == ~0ull) continue;
    if (out && n < max_records) out[n] = r;
    ++n;
  }
  *n_out = n;
  return SWARM_OK;
}

swarm_status swarm_trace_events(swarm_t h, swarm_event* out, int32_t* counts) {
  if (!h || !out || !counts) return fail(SWARM_ERR_INVALID_ARG, "NULL argument");
  if (h->in_flight) return busy();
  if (!h->have_run || !h->traced) return fail(SWARM_ERR_STATE, "no traced run");
  hipError_t e = hipMemcpyAsync(out, h->trace_out.p, static_cast<size_t>(h->n_trace) * h->max_events * sizeof(swarm_event),
                                hipMemcpyDeviceToHost, h->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(counts, h->trace_count.p, h->n_trace * sizeof(int32_t), hipMemcpyDeviceToHost, h->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  if (e != hipSuccess) return hip_fail(e, "copying trace");
  return SWARM_OK;
}

swarm_status swarm_tables(swarm_t h, int32_t* grid_size, int32_t* n_channels, double* nodes, double* cum,
                          double* majorant) {
  if (!h) return fail(SWARM_ERR_INVALID_ARG, "handle is NULL");
  if (grid_size) *grid_size = h->desc.G;
  if (n_channels) *n_channels = h->desc.nc;
  if (majorant) *majorant = h->desc.majorant;
  hipError_t e = hipSuccess;
  if (nodes) e = hipMemcpyAsync(nodes, h->desc.nodes, h->desc.G * sizeof(double), hipMemcpyDeviceToHost, h->stream);
  if (e == hipSuccess && cum)
    e = hipMemcpyAsync(cum, h->desc.cum_cm, static_cast<size_t>(h->desc.G) * h->desc.nc * sizeof(double),
                       hipMemcpyDeviceToHost, h->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  if (e != hipSuccess) return hip_fail(e, "copying tables");
  return SWARM_OK;
}

swarm_status swarm_last_timing(swarm_t h, double* kernel_ms, double* total_ms) {
  if (!h) return fail(SWARM_ERR_INVALID_ARG, "handle is NULL");
  if (h->in_flight) return busy();
  if (!h->have_run) return fail(SWARM_ERR_STATE, "no completed run");
  if (kernel_ms) *kernel_ms = h->kernel_ms;
  if (total_ms) *total_ms = h->total_ms;
  return SWARM_OK;
}

swarm_status swarm_last_launches(swarm_t h, int64_t* launches, int64_t* parked) {
  if (!h) return fail(SWARM_ERR_INVALID_ARG, "handle is NULL");
  if (h->in_flight) return busy();
  if (!h->have_run) return fail(SWARM_ERR_STATE, "no completed run");
  if (launches) *launches = h->n_launches;
  if (parked) *parked = h->n_parked;
  return SWARM_OK;
}

swarm_status swarm_last_team(swarm_t h, int32_t* lanes) {
  if (!h || !lanes) return fail(SWARM_ERR_INVALID_ARG, "NULL argument");
  if (h->in_flight) return busy();
  if (!h->have_run) return fail(SWARM_ERR_STATE, "no completed run");
  *lanes = h->team_lanes;
  return SWARM_OK;
}

}  // extern "C"
