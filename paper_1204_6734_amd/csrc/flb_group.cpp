// flb_group.cpp — lattices and ensembles.  Both are a "group" of slots that
// share a stream, a device clock and one batched step launch per step; a
// lattice is a group of one slot (and is the only kind with the
// structure-factor pipeline).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <numeric>
#include <vector>

#include "flb.h"
#include "flb_group.hpp"
#include "flb_runtime.hpp"

namespace flb {

#define HIPC(expr)                                    \
  do {                                                \
    hipError_t e_ = (expr);                           \
    if (e_ != hipSuccess) return hip_fail(e_, #expr); \
  } while (0)

static size_t storage_size(int storage) { return storage == 0 ? sizeof(double) : sizeof(float); }

// Lay out every device array of the group in `a` (a.base may be null to
// size it).
void Group::layout(Arena& a, bool second) {
  const int n = (int)P.size();
  d_slots = a.take<SlotDesc>(n);
  d_prefix = a.take<int>(n + 2);
  if (plain_tiles) {
    d_plain = a.take<SlotDesc>(n);
    d_plain_prefix = a.take<int>(n + 2);
  }
  d_clock = a.take<uint64_t>(1);
  d_err = a.take<int>(n);
  d_err_step = a.take<unsigned long long>(n);
  d_open = a.take<double>((size_t)(1 + kFoldRows) * kNStat);
  d_B = a.take<double>(81);
  d_mode = a.take<double2>(kModeBlocks);
  d_close = a.take<double*>(2 * (size_t)n);
  pop.resize(n);
  d_partials.assign(n, nullptr);
  d_records.assign(n, nullptr);
  size_t max_sites = 0;
  for (int s = 0; s < n; ++s) {
    const size_t N = (size_t)P[s].nx * P[s].ny;
    max_sites = std::max(max_sites, N);
    pop[s] = a.take<char>(population_elems(P[s].nx, P[s].ny) * storage_size(storage));
    if (P[s].sample_every > 0) {
      d_partials[s] = a.take<double>((size_t)hdesc[s].ntiles * kNStat);
      d_records[s] = a.take<double>((size_t)kMaxTimeBlocks * kNStat);
    }
  }
  // staging for host I/O, one band of rows at a time
  int maxnx = 0, maxny = 0;
  for (auto& p : P) {
    maxnx = std::max(maxnx, p.nx);
    maxny = std::max(maxny, p.ny);
  }
  band_rows = std::max(1, std::min(maxny, (int)((1u << 22) / (unsigned)maxnx)));
  d_io = a.take<double>((size_t)9 * band_rows * maxnx);
  if (n == 1 && P[0].sk_every > 0) {
    const size_t N = max_sites, cplx = 2 * storage_size(storage);
    d_z = a.take<char>(2 * N * cplx);
    d_zt = a.take<char>(2 * N * cplx);
    d_skacc = a.take<double>(5 * sk_half());
    d_twx = a.take<char>(P[0].nx * cplx);
    d_twy = a.take<char>(P[0].ny * cplx);
  }
  // the several-step kernel's second population buffer, all slots together
  pop2 = nullptr;
  if (second)
    for (int s = 0; s < n; ++s) {
      char* p = a.take<char>(population_elems(P[s].nx, P[s].ny) * storage_size(storage));
      if (s == 0) pop2 = p;
      hdesc[s].pop2 = p;
    }
}

int Group::init(const flb_params* ps, int n, void* stream, void* dev_buf, size_t dev_bytes) {
  if (n <= 0) return set_error(FLB_E_ARG, "need at least one lattice");
  for (int s = 0; s < n; ++s) {
    const int rc = check_params(&ps[s]);
    if (rc != FLB_OK) return rc;
    if (ps[s].nx != ps[0].nx || ps[s].ny != ps[0].ny || ps[s].precision != ps[0].precision ||
        ps[s].basis != ps[0].basis)
      return set_error(FLB_E_ARG, "ensemble members must share nx, ny, precision and basis");
    if (n > 1 && ps[s].sk_every > 0)
      return set_error(FLB_E_ARG, "structure factors are available for single lattices only");
  }
  P.assign(ps, ps + n);
  storage = ps[0].precision == FLB_FP64 ? 0 : 1;
  basis = ps[0].basis;
  compute = 1;
  for (int s = 0; s < n; ++s) compute = std::min(compute, compute_precision(&ps[s]));
  // launch classes: FP32-compute members first, then FP64-compute members
  corder.clear();
  nclass = 0;
  for (int cc : {1, 0}) {
    const int first = (int)corder.size();
    for (int s = 0; s < n; ++s)
      if (compute_precision(&ps[s]) == cc) corder.push_back(s);
    if ((int)corder.size() > first) {
      ccompute[nclass] = cc;
      cfirst[nclass] = first;
      ccount[nclass] = (int)corder.size() - first;
      ++nclass;
    }
  }
  hdesc.assign(n, SlotDesc{});
  prefix.assign(n + 1, 0);
  sample_intervals.clear();
  for (int s = 0; s < n; ++s) {
    const uint64_t every = (uint64_t)ps[s].sample_every;
    if (every && std::find(sample_intervals.begin(), sample_intervals.end(), every) ==
                     sample_intervals.end())
      sample_intervals.push_back(every);
    fill_slot(&ps[s], &hdesc[s]);
    prefix[s + 1] = prefix[s] + hdesc[s].ntiles;
  }
  total_tiles = prefix[n];
  // The members' shape is one that suits the launches of several steps, which a
  // group of this size does not take, and the order of the sums, which are the
  // same for a member as alone, hangs on it.  Beyond the 256 MiB last-level
  // cache the steps without sums are faster in 256 x 1 tiles (us a step, 64 x 4
  // -> 256 x 1: 128 x 256^2 108.2 -> 104.4, 160 x 1000x60 132 -> 125, 600 x 256x100
  // 206 -> 199; 64 x 256^2, 151 MiB, 47.7 -> 47.6); those with sums are not (129
  // and 129).
  if (small_lattice_tiles(ps[0]) &&
      (double)population_elems(ps[0].nx, ps[0].ny) * n * sizeof(float) > 256.0 * (1 << 20)) {
    SlotDesc d = hdesc[0];
    set_tiles(&d, 1);
    plain_tiles = d.ntiles;
  }
  int lds = 0, cus = 0;
  HIPC(hipGetDevice(&device));
  HIPC(hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, device));
  HIPC(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device));
  max_lds = (size_t)lds;
  Arena sizing;
  layout(sizing);
  need_bytes = sizing.used + 256;
  bool second = false;
  if (dev_buf) {
    if (dev_bytes < need_bytes)
      return set_error(FLB_E_ARG, "device buffer too small: %zu < %zu bytes", dev_bytes,
                       need_bytes);
    dev = dev_buf;
    own_mem = false;
  } else {
    hipError_t e = hipErrorOutOfMemory;
    plan_multi(cus);
    if (!passes_pay()) multi_max = march_rows = 0;
    if (multi_max) {
      Arena both;
      layout(both, true);
      second = take_second(both.used + 256 - need_bytes);
      if (second) e = hipMalloc(&dev, both.used + 256);
      if (second && e != hipSuccess) {
        (void)hipGetLastError();
        second_bytes.give();
        second = false;  // one step per launch needs less
      }
      if (second) need_bytes = both.used + 256;
    }
    if (!second) {
      multi_max = march_rows = 0;
      e = hipMalloc(&dev, need_bytes);
    }
    if (e != hipSuccess) {
      dev = nullptr;
      return set_error(FLB_E_OOM, "hipMalloc(%zu): %s", need_bytes, hipGetErrorString(e));
    }
    own_mem = true;
  }
  Arena a;
  a.base = (char*)(((uintptr_t)dev + 255) & ~(uintptr_t)255);
  layout(a, second);
  if (stream) {
    st = (hipStream_t)stream;
    own_stream = false;
  } else {
    HIPC(hipStreamCreateWithFlags(&st, hipStreamNonBlocking));
    own_stream = true;
  }
  if (d_skacc && (!sk_transform_supported(P[0].nx, storage, max_lds) ||
                  !sk_transform_supported(P[0].ny, storage, max_lds)))
    return set_error(FLB_E_ARG,
                     "structure factors need sides that are powers of two up to %d (FP64) or "
                     "%d (FP32) or at most %d",
                     (int)(max_lds / sizeof(double2)), (int)(max_lds / sizeof(float2)),
                     kMaxDirectDft);
  if (multi_max && !march_rows)
    for (int c = 0; c < nclass; ++c)
      HIPC(multi_prepare(storage, ccompute[c], basis, P[0].nx, multi_max, max_lds));
  launch = tuned_launch(*this);
  // per-slot pointers and measurement bases
  mt0.assign(n, std::vector<double>(81));
  stats.assign(n, Stats{});
  for (int s = 0; s < n; ++s) {
    hdesc[s].pop = pop[s];
    hdesc[s].partials = d_partials[s];
    hdesc[s].skz = d_z;
    hdesc[s].err = d_err + s;
    hdesc[s].err_step = d_err_step + s;
    hdesc[s].t0 = 0;
    hdesc[s].tend = 0x7FFFFFFFFFFFFFFFull;  // never
    fnorm_rows(ps[s].ux0, ps[s].uy0, mt0[s].data());
    stats[s].reset(ps[s].block_steps);
  }
  {
    std::vector<SlotDesc> dev_desc(n);
    std::vector<int> dev_prefix;
    for (int c = 0; c < nclass; ++c) {
      int acc = 0;
      dev_prefix.push_back(0);
      for (int j = 0; j < ccount[c]; ++j) {
        const int s = corder[cfirst[c] + j];
        dev_desc[cfirst[c] + j] = hdesc[s];
        acc += hdesc[s].ntiles;
        dev_prefix.push_back(acc);
      }
      ctiles[c] = acc;
    }
    HIPC(hipMemcpy(d_slots, dev_desc.data(), n * sizeof(SlotDesc), hipMemcpyHostToDevice));
    if (plain_tiles) {
      std::vector<int> plain_prefix;
      for (int c = 0; c < nclass; ++c)
        for (int j = 0; j <= ccount[c]; ++j) plain_prefix.push_back(j * plain_tiles);
      for (SlotDesc& d : dev_desc) set_tiles(&d, 1);
      HIPC(hipMemcpy(d_plain, dev_desc.data(), n * sizeof(SlotDesc), hipMemcpyHostToDevice));
      HIPC(hipMemcpy(d_plain_prefix, plain_prefix.data(), plain_prefix.size() * sizeof(int),
                     hipMemcpyHostToDevice));
    }
    std::vector<double*> close(2 * (size_t)n);
    for (int s = 0; s < n; ++s) {
      close[s] = d_partials[s];
      close[n + s] = d_records[s];
    }
    HIPC(hipMemcpy(d_close, close.data(), close.size() * sizeof(double*), hipMemcpyHostToDevice));
    HIPC(hipMemcpy(d_prefix, dev_prefix.data(), dev_prefix.size() * sizeof(int),
                   hipMemcpyHostToDevice));
  }
  HIPC(hipMemsetAsync(d_clock, 0, sizeof(uint64_t), st));
  HIPC(hipMemsetAsync(d_err, 0, n * sizeof(int), st));
  HIPC(hipMemsetAsync(d_err_step, 0xFF, n * sizeof(unsigned long long), st));
  for (int s = 0; s < n; ++s) {
    if (d_partials[s]) {
      HIPC(launch_fill(d_partials[s], (size_t)hdesc[s].ntiles * kNStat, 0.0, st));
      HIPC(launch_fill(d_records[s], (size_t)kMaxTimeBlocks * kNStat, 0.0, st));
    }
  }
  if (d_skacc) {
    const int nx = P[0].nx, ny = P[0].ny;
    HIPC(launch_fill(d_skacc, 5 * sk_half(), 0.0, st));
    // twiddles exp(-2 pi i k / n), k < n, in the storage precision
    for (int dim = 0; dim < 2; ++dim) {
      const int m = dim == 0 ? nx : ny;
      std::vector<double> tw(2 * (size_t)m);
      std::vector<float> twf(2 * (size_t)m);
      for (int k = 0; k < m; ++k) {
        const double ph = -2.0 * M_PI * (double)k / (double)m;
        tw[2 * k] = std::cos(ph);
        tw[2 * k + 1] = std::sin(ph);
        twf[2 * k] = (float)tw[2 * k];
        twf[2 * k + 1] = (float)tw[2 * k + 1];
      }
      const void* src = storage == 0 ? (const void*)tw.data() : (const void*)twf.data();
      HIPC(hipMemcpy(dim == 0 ? d_twx : d_twy, src, 2 * (size_t)m * storage_size(storage),
                     hipMemcpyHostToDevice));
    }
    HIPC(sk_prepare(max_lds));
  }
  for (int s = 0; s < n; ++s) {
    const flb_params& p = P[s];
    const double mu = p.init == FLB_INIT_THERMAL ? 3.0 * p.kT : 0.0;
    for (int y0 = 0; y0 < p.ny; y0 += band_rows) {
      const int rows = std::min(band_rows, p.ny - y0);
      HIPC(launch_init(storage, pop[s], hdesc[s].pitch, nullptr, nullptr, nullptr, p.rho0, p.ux0, p.uy0,
                       slot_shift(hdesc[s]), p.nx, p.ny, mu, hdesc[s].k0, hdesc[s].k1, 0, y0, rows,
                       st));
    }
  }
  t = 0;
  HIPC(hipStreamSynchronize(st));
  return FLB_OK;
}

Group::~Group() {
  if (st) (void)wait();
  for (auto& e : events) {
    (void)hipEventDestroy(e.first);
    (void)hipEventDestroy(e.second);
  }
  drop_graph();
  for (int i = 0; i < kMaxBranches; ++i) {
    if (joined[i]) (void)hipEventDestroy(joined[i]);
    if (branch[i]) (void)hipStreamDestroy(branch[i]);
  }
  if (own_mem && dev) (void)hipFree(dev);
  if (own_stream && st) (void)hipStreamDestroy(st);
}

bool Group::sample_due(int s, uint64_t tt) const {
  const flb_params& p = P[s];
  return p.sample_every > 0 && tt % (uint64_t)p.sample_every == 0;
}

bool Group::sk_due(int s, uint64_t tt) const {
  const flb_params& p = P[s];
  return d_skacc && p.sk_every > 0 && tt % (uint64_t)p.sk_every == 0;
}

// Whether every slot closes a time block after the sample of time tt, all
// at the same record index, with no record merge first and one tile count:
// an ensemble whose replicas sample alike.  Then one batched launch closes
// them all, each with the additions of its own close.
bool Group::lockstep_close(uint64_t tt) const {
  const int n = (int)P.size();
  if (n < 2) return false;
  for (int s = 0; s < n; ++s)
    if (!sample_due(s, tt) || !stats[s].plain_close_next() || stats[s].nb != stats[0].nb ||
        hdesc[s].ntiles != hdesc[0].ntiles)
      return false;
  return true;
}

// Work after the step kernel of time tt: structure-factor transform and
// time-block bookkeeping.  After a graph replay the transforms of the
// chunk's steps ran inside the graph (replayed = true): only the counts and
// the time-block closes remain.
int Group::after_step(uint64_t tt, bool replayed) {
  const int n = (int)P.size();
  for (int s = 0; s < n; ++s) {
    if (sk_due(s, tt)) {
      if (!replayed)
        HIPC(launch_sk_sample(storage, d_z, d_zt, d_skacc, P[s].nx, P[s].ny, d_twx, d_twy,
                              max_lds, st));
      nsk += 1;
    }
  }
  if (lockstep_close(tt)) {
    uint64_t b = 0;
    for (int s = 0; s < n; ++s) b = stats[s].close_counted((uint64_t)P[s].nx * P[s].ny);
    HIPC(launch_close_block_many(d_close, d_close + n, (size_t)b * kNStat, n, hdesc[0].ntiles,
                                 st));
    return FLB_OK;
  }
  for (int s = 0; s < n; ++s)
    if (sample_due(s, tt))
      HIPC(stats[s].after_sample((uint64_t)P[s].nx * P[s].ny, d_partials[s], hdesc[s].ntiles,
                                 d_records[s], st));
  return FLB_OK;
}

// The step launches of one step: one per compute class, of all members or of
// one of `parts` equal shares of them (members of one tile count: the prefix
// sums of a share are the first ones) on stream q.
hipError_t Group::launch_classes(uint32_t k, bool sample, int odd, LaunchCfg c, int part,
                                 int parts, hipStream_t q) {
  for (int i = 0; i < nclass; ++i) {
    const int a = ccount[i] * part / parts, b = ccount[i] * (part + 1) / parts;
    if (a == b) continue;
    const bool plain = plain_tiles && !sample;
    const int tiles = plain ? (b - a) * plain_tiles
                            : (parts == 1 ? ctiles[i] : (b - a) * hdesc[0].ntiles);
    const hipError_t e =
        launch_step(storage, ccompute[i], basis, sample, odd,
                    (plain ? d_plain : d_slots) + cfirst[i] + a,
                    (plain ? d_plain_prefix : d_prefix) + cfirst[i] + i, b - a, tiles, d_clock, k,
                    c, q);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
hipError_t Group::launch_classes(uint32_t k, bool sample, int odd, LaunchCfg c) {
  return launch_classes(k, sample, odd, c, 0, 1, st);
}

// fn() enqueues `steps` steps; with profiling on, between two events.
template <typename Fn>
int Group::profiled(Fn fn, uint64_t steps) {
  if (profiling) {
    std::pair<hipEvent_t, hipEvent_t> ev;
    HIPC(hipEventCreate(&ev.first));
    HIPC(hipEventCreate(&ev.second));
    HIPC(hipEventRecord(ev.first, st));
    HIPC(fn());
    HIPC(hipEventRecord(ev.second, st));
    events.push_back(ev);
    prof_launches += steps;
    return FLB_OK;
  }
  HIPC(fn());
  return FLB_OK;
}

// A captured chunk of graph_chunk steps can be replayed at every time that
// is a multiple of graph_chunk when each slot's sampling and structure-factor
// intervals divide the chunk: the pattern of sampled steps inside a chunk is
// then the same every time.
bool Group::graph_friendly() const {
  if (graph_chunk <= 0) return false;
  for (auto& p : P) {
    if (p.sample_every > 0 && graph_chunk % p.sample_every != 0) return false;
    if (d_skacc && p.sk_every > 0 && graph_chunk % p.sk_every != 0) return false;
  }
  return true;
}

// Steps from time tt (up to which the samples are counted) until (and
// including) the first step after tt + skip whose sample closes a time block
// of some slot; replays and several-step launches must not straddle one.
uint64_t Group::steps_to_close(uint64_t tt, uint64_t skip) const {
  uint64_t m = ~0ull;
  for (int s = 0; s < (int)P.size(); ++s) {
    const uint64_t se = (uint64_t)P[s].sample_every, len = stats[s].tb_len;
    if (se == 0 || len == 0) continue;
    const uint64_t left = len - stats[s].tb_fill;       // samples to the close
    const uint64_t first = (tt + se - 1) / se * se;     // next sampled time
    uint64_t r = first + (left - 1) * se - tt + 1;
    while (r <= skip) r += len * se;
    m = std::min(m, r);
  }
  return m;
}

// ------------------------------------------------- several steps per launch
// The numbers of steps that launches take.  Several steps pay while a step is
// held by latency, that is while the chip is not full: at one tile per
// workgroup (the halo is cheapest to recompute when nothing else wants the
// SIMDs; two tiles measured slower), up to one workgroup per CU.  Measured (us a step, one step per launch -> this; without
// / with sums of every step): FP32 21^2 2.9 -> 1.8 / 4.0 -> 2.2, 64^2 2.9 ->
// 2.3 / 4.1 -> 2.9, 256^2 (256 tiles) 3.2 -> 2.8 / 4.1 -> 3.4, but 256 x 320
// (320 tiles) 3.6 -> 4.7 / 4.7 -> 6.3.  Lattices of two or more rows per
// wavefront have short workgroups, two of which share a CU (64 x 21^2, 384
// tiles: 3.8 -> 2.3 / 4.8 -> 3.1), and take six steps as well as four.  FP64
// collisions gain on those only (21^2 3.7 -> 2.5 / 4.9 -> 3.5, 32^2 3.6 -> 3.1
// / 4.9 -> 4.2; 64^2 3.7 -> 3.9 / 4.9 -> 5.5): their halo costs more than the
// launches saved.  They take six steps with four or more rows per wavefront
// (four -> six: 12^2 2.43 -> 2.26 / 3.23 -> 2.90, 16^2 2.45 -> 2.28; 21^2 2.51
// -> 2.64).
// A program may step several lattices side by side, each on its own stream,
// and the recomputed halo then takes time from the others once they fill the
// chip together: so the wavefronts of a launch are bounded by what three side
// by side still gain with, and a launch takes fewer steps, or one, above that.
// Three FP32 lattices, us a step of all: 256^2 plain 4.2 one step a launch, 4.3
// two (7 wavefronts a CU), 6.6 four (11); with sums 256 x 128 6.3 -> 5.7, 256 x
// 160 9.7 -> 10.5, 256^2 6.9 -> 10.0; 24 x 32^2 with sums 5.2 -> 4.8 (8.3
// wavefronts a CU), 32 x 32^2 5.3 -> 6.4 (11); FP64 16 x 32^2 4.8 -> 4.2 (4.5),
// 40 x 21^2 5.3 -> 4.1 two steps (3.8), 6.4 four (6.6), 32 x 32^2 5.5 -> 6.5
// two (5), 8.3 four (9).
void Group::plan_multi(int cus) {
  multi_max = 0;
  std::fill(&multi_takes[0][0], &multi_takes[0][0] + 2 * (kMultiMaxSteps + 1), false);
  march_rows = plan_march(cus);
  if (march_rows) {
    multi_takes[0][2] = true;  // steps without sums only
    multi_max = 2;
    return;
  }
  const int nx = P[0].nx;
  const bool narrow = nx <= kTileX / 2;
  if (hdesc[0].wide || (compute == 0 && !narrow)) return;
  if (total_tiles > (narrow && compute == 1 ? 2 * cus : cus)) return;
  const int most =
      narrow && (compute == 1 || nx <= kTileX / 4) && total_tiles <= cus ? 6 : 4;
  for (int sample = 0; sample < 2; ++sample)
    for (int K = 2; K <= most; K += 2) {
      if (!multi_fits(storage, compute, sample != 0, nx, K, max_lds)) continue;
      const double waves = (double)total_tiles * multi_waves(compute, sample != 0, nx, K);
      if (sample && !narrow ? 2 * total_tiles > cus
                            : waves > (compute == 0 ? 4.9 : sample ? 8.3 : 7.0) * cus)
        continue;
      multi_takes[sample][K] = true;
      multi_max = std::max(multi_max, K);
    }
}

// Rows a wavefront of step_march_kernel takes, 0 where one step per launch is
// the better one.  Two steps per pass over memory halve the traffic and cost
// (64/62)(1 + 1/H) of the arithmetic, so they pay where the FP32 arithmetic is
// the smaller part: in the Hermite basis where the populations exceed the 32 MiB
// of the XCDs' L2 caches, in the others (twice the arithmetic) where they exceed
// the 256 MiB last-level cache.  Not in FP64: f-norm lattices run 8 % faster in
// the cache than beyond it (40.9 GLUPS at 1792^2, 220 MiB, 37.4-37.6 from 3072^2
// on; mixed relaxation times 39.4 and 36.2-36.5), which the 6.5 % of halo sites
// would take; the Hermite basis was not tried.  us a step, one step per launch ->
// this kernel:
//   f-norm   2560^2 (225 MiB) 71 -> 78, 2003x4001 (275) 95.5 -> 96.4, 2900^2
//            (289) 105 -> 100, 3072^2 (324) 116 -> 107, 8192^2 845 -> 694
//   Hermite  1003x601 (21) 7.7 -> 8.1, 1024^2 (36) 13.8 -> 11.3, 2048^2 43.8 ->
//            33.9, 8192^2 826 -> 507
// Narrow members waste lanes of their last strip (f-norm): 200^2 x 256 (78 %
// used) 160 -> 138, 256^2 x 256 (80 %) 223 -> 211, 128^2 x 1000 (67 %) 217 ->
// 239.  Rows: more share the first and last among themselves, fewer keep more
// wavefronts in flight and the rows of neighbouring bands in the cache.  f-norm:
// 32 once that is four rounds of the 16 wavefronts a compute unit holds (8192^2
// 703 -> 694), 16 below (4096^2 187 -> 183, 2816^2 92 -> 91).  Hermite: 8 once
// that is one round (8192^2: 529, 507, 544 at 4, 8, 16; 1536^2: 19.7, 18.4,
// 21.9), 4 below (1024^2: 11.3, 12.3).
int Group::plan_march(int cus) const {
  const int nx = P[0].nx, ny = P[0].ny, n = (int)P.size();
  if (storage != 1 || compute != 1) return 0;
  const bool hermite = basis == FLB_BASIS_HERMITE;
  const double bytes = (double)nx * ny * n * 36.0, mib = 1 << 20;
  if (bytes < (hermite ? 32 : 300) * mib) return 0;
  const int strips = (nx + kMarchCols - 1) / kMarchCols;
  if (4 * nx < 3 * 64 * strips) return 0;
  const int rows = hermite ? 8 : 32;
  const double waves = (double)strips * ((ny + rows - 1) / rows) * n;
  return waves >= (hermite ? 16.0 : 64.0) * cus ? rows : rows / 2;
}

// Whether a second population buffer of this size is taken: where all of the
// process's on the device then hold at most a fifteenth of what stays free.  So a
// program that fills the memory, with one lattice or with thousands of small ones,
// holds at least fifteen sixteenths of what it would, also where others hold most
// of it; and memory in use takes the launches of several steps from a lattice only
// where its buffer would be a large part of the rest (16384 x 16384 takes twice 9.7
// of 288 GB).
bool Group::take_second(size_t bytes) {
  size_t freeb = 0, total = 0;
  if (hipMemGetInfo(&freeb, &total) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  if (freeb < need_bytes + bytes) return false;
  return second_bytes.take(device, bytes, (freeb - need_bytes - bytes) / 15);
}

// Largest launch from the even time tt within `lim` steps that holds no
// structure-factor step but its first.
int Group::pass_steps(uint64_t tt, uint64_t lim) const {
  if (const uint64_t sk = (uint64_t)sk_interval()) lim = std::min(lim, sk - tt % sk);
  for (int K = multi_max; K >= 2; K -= 2)
    if ((uint64_t)K <= lim && multi_takes[pass_samples(tt, K)][K]) return K;
  return 0;
}

// Whether a launch of K steps from time tt takes the variant with sums.
bool Group::pass_samples(uint64_t tt, int K) const {
  const uint64_t sk = (uint64_t)sk_interval();
  if (sk && tt % sk == 0) return true;
  for (uint64_t se : sample_intervals)
    if ((tt + se - 1) / se * se < tt + (uint64_t)K) return true;
  return false;
}

// The next two launches of several steps from time tt (pop -> pop2 -> pop:
// outside a pair the state is always in the first buffer), within `left`
// steps and with time blocks closing after a launch at most.  kb = 0: none.
void Group::pass_pair(uint64_t tt, uint64_t left, bool closes, int* ka, int* kb) const {
  *ka = *kb = 0;
  if (!multi_max || forced_launch || (tt & 1)) return;
  const uint64_t m = closes ? steps_to_close(tt, 0) : ~0ull;
  for (int K = pass_steps(tt, std::min(left, m)); K >= 2; K -= 2) {
    if (!multi_takes[pass_samples(tt, K)][K]) continue;
    const uint64_t m2 = closes ? steps_to_close(tt, (uint64_t)K) - (uint64_t)K : ~0ull;
    *ka = K;
    *kb = pass_steps(tt + (uint64_t)K, std::min(left - (uint64_t)K, m2));
    if (*kb) return;
  }
}

// Share of the first `steps` steps (0: of some periods of the sampling) that
// launches of several steps take, time blocks aside.
double Group::pass_share(uint64_t steps) const {
  if (!multi_max) return 0.0;
  if (!steps) {
    uint64_t period = 2;
    for (uint64_t e : sample_intervals) period = std::min<uint64_t>(std::lcm(period, e), 2048);
    if (const uint64_t sk = (uint64_t)sk_interval())
      period = std::min<uint64_t>(std::lcm(period, sk), 2048);
    steps = (96 + period - 1) / period * period;
  }
  uint64_t taken = 0;
  for (uint64_t tt = 0; tt < steps;) {
    int pass[2];
    pass_pair(tt, steps - tt, false, &pass[0], &pass[1]);
    const uint64_t k = pass[1] ? (uint64_t)(pass[0] + pass[1]) : 0;
    taken += k;
    tt += k ? k : 1;
  }
  return (double)taken / (double)steps;
}

// Whether what was planned pays with the members' sampling.  Where only steps
// without sums are taken together, a lattice that samples every step has none
// and needs no second buffer.  In the f-norm bases, strips that use less than
// nine tenths of their lanes lose in part of the steps more than they gain in
// the others below 400 MiB, and beyond with few such steps (us a step, one step
// per launch -> passes; sums every 5, 8, 10, no steps: 160 x 256^2, 360 MiB,
// 139.0 -> 143.7, 137.1 -> 141.6, 136.7 -> 138.1, 134.0 -> 133.2; 200 x 256^2, 450
// MiB, 175.6 -> 178.8, 173.8 -> 176.0, 173.3 -> 170.3, 170.7 -> 164.2).  Wider strips gain throughout (8192^2 873 -> 837, 859
// -> 818, 856 -> 764; 3072^2 121 -> 119, 119 -> 117, 119 -> 113), and so does the
// Hermite basis (64 x 160^2 20.3 -> 18.7, 20.2 -> 18.1, 20.1 -> 16.6).
bool Group::passes_pay() const {
  const double share = pass_share();
  if (!march_rows || basis == FLB_BASIS_HERMITE) return share > 0;
  const int nx = P[0].nx, strips = (nx + kMarchCols - 1) / kMarchCols;
  const double bytes = (double)population_elems(nx, P[0].ny) * P.size() * sizeof(float);
  if (10 * nx < 9 * 64 * strips && (bytes < 400.0 * (1 << 20) || share < 0.6)) return false;
  return share > 0;
}

// One launch of K steps from time tt (step index k of the device clock).
hipError_t Group::launch_pass(uint32_t k, uint64_t tt, int K, int flip) {
  if (march_rows)
    return launch_step_march(basis, d_slots, (int)P.size(), P[0].nx, P[0].ny, march_rows, flip,
                             d_clock, k, st);
  const bool sample = pass_samples(tt, K);
  for (int i = 0; i < nclass; ++i) {
    const hipError_t e =
        launch_step_multi(storage, ccompute[i], basis, sample, d_slots + cfirst[i], ccount[i],
                          P[0].nx, P[0].ny, K, flip, d_clock, k, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Branches of a captured chunk.  Members do not depend on each other, so two
// halves can advance side by side: while one half's step ends and its next one
// starts, the other's fills the chip.  A branch costs the replay 7.8 us a step
// at least, so the chunk stays one chain below the tiles whose step takes
// about that (FP32 2048 tiles of 256 sites, FP64 1024).  Measured (us a step,
// one branch -> two; more gained nothing): FP32 1024 tiles 5.7 -> 7.8, 2048 9.2
// -> 8.1, 4096 (64 x 128^2) 16.2 -> 13.5, 16384 51.6 -> 46.9, 32768 101.5 ->
// 100.1; FP64 512 tiles 5.3 -> 7.9, 1024 9.7 -> 8.4, 2048 17.8 -> 13.8, 16384
// 116.5 -> 112.6.  Ensembles stepped side by side on streams of their own fill
// the chip by themselves, and the second branch costs there until their
// populations outgrow the last-level cache; so beside other work it is taken
// from 16384 tiles on (FP64 8192).  us a step of all, one branch -> two:
//                two at once                three at once
//   FP32  2048   12.2 -> 15.2               18.8 -> 22.9
//         4096   23.7 -> 27.4               34.9 -> 42.0
//         8192   45.0 -> 48.4               66.9 -> 77.1
//        12288   67.0 -> 70.7, with sums    115.6 -> 109.7, with sums
//                76.4 -> 73.0               117.1 -> 112.4
//        16384   98.0 -> 89.3               158.8 -> 137.5
//   FP64  1024   14.1 -> 16.7               20.3 -> 25.0
//         4096   51.4 -> 53.2               76.5 -> 84.8
//         8192   112.2 -> 103.7             171.6 -> 160.3
// Alone means at this replay and the one before: of ensembles stepped in turn
// and then waited for, the first to go on is not taken for a lone one.
// Two steps per pass over memory and two branches exclude each other: the passes
// are taken where they cover half of the chunk's steps, in the Hermite basis
// always (us a step, passes / two branches; sums every 5, 10, no steps: Hermite
// 64 x 160^2 18.7 / 18.8, 16.7 / 18.6, 15.4 / 18.3; f-norm 9 x 1003^2 118.8 /
// 114.5, 112.2 / 110.5, 106.6 / 108.2, 256 x 200^2 163 / 179, 145 / 179, 136 /
// 158).
int Group::graph_branches(bool alone) const {
  if (P.size() < 2 || d_skacc || forced_launch) return 1;
  if (!two_branches(compute, total_tiles, alone)) return 1;
  const double share = pass_share((uint64_t)graph_chunk);
  if (share > 0 && (!march_rows || basis == FLB_BASIS_HERMITE || share >= 0.5)) return 1;
  for (auto& h : hdesc)
    if (h.ntiles != hdesc[0].ntiles) return 1;
  return 2;
}

int Group::abandon_capture(hipError_t e) {
  hipGraph_t g = nullptr;
  (void)hipStreamEndCapture(st, &g);
  if (g) (void)hipGraphDestroy(g);
  return hip_fail(e, "capture step");
}

int Group::capture_graph(int parts) {
  if (graph_exec[parts - 1]) return FLB_OK;
  if (parts > 1) {
    OnDevice on(device);
    if (!joined[0]) HIPC(hipEventCreateWithFlags(&joined[0], hipEventDisableTiming));
    for (int i = 1; i < parts; ++i) {
      if (!branch[i]) HIPC(hipStreamCreateWithFlags(&branch[i], hipStreamNonBlocking));
      if (!joined[i]) HIPC(hipEventCreateWithFlags(&joined[i], hipEventDisableTiming));
    }
  }
  HIPC(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
  if (parts > 1) {
    hipError_t e = hipEventRecord(joined[0], st);
    for (int i = 1; i < parts && e == hipSuccess; ++i)
      e = hipStreamWaitEvent(branch[i], joined[0], 0);
    if (e != hipSuccess) return abandon_capture(e);
  }
  graph_passed[parts - 1] = 0;
  for (int k = 0; k < graph_chunk; ++k) {
    int pass[2];
    pass_pair((uint64_t)k, (uint64_t)(graph_chunk - k), false, &pass[0], &pass[1]);
    if (pass[1] && parts == 1) {
      hipError_t e = hipSuccess;
      for (int i = 0; i < 2 && e == hipSuccess; ++i) {
        e = launch_pass((uint32_t)k, (uint64_t)k, pass[i], i);
        if (e == hipSuccess && sk_due(0, (uint64_t)k))
          e = launch_sk_sample(storage, d_z, d_zt, d_skacc, P[0].nx, P[0].ny, d_twx, d_twy,
                               max_lds, st);
        k += pass[i];
        graph_passed[parts - 1] += (uint64_t)pass[i];
      }
      if (e != hipSuccess) return abandon_capture(e);
      --k;  // the loop's own step
      continue;
    }
    // replays start at multiples of graph_chunk (even), so step k of a chunk
    // has parity k & 1 and a slot samples there iff k is a multiple of its
    // interval; a structure-factor step also takes the sampling variant (it
    // writes the fields) and is followed by its transform
    bool sample = false;
    for (int s = 0; s < (int)P.size(); ++s)
      sample |= sample_due(s, (uint64_t)k) || sk_due(s, (uint64_t)k);
    hipError_t e = hipSuccess;
    for (int i = 0; i < parts && e == hipSuccess; ++i)
      e = launch_classes((uint32_t)k, sample, k & 1, launch, i, parts, i ? branch[i] : st);
    for (int s = 0; s < (int)P.size() && e == hipSuccess; ++s)
      if (sk_due(s, (uint64_t)k))
        e = launch_sk_sample(storage, d_z, d_zt, d_skacc, P[s].nx, P[s].ny, d_twx, d_twy,
                             max_lds, st);
    if (e != hipSuccess) return abandon_capture(e);
  }
  for (int i = 1; i < parts; ++i) {
    hipError_t e = hipEventRecord(joined[i], branch[i]);
    if (e == hipSuccess) e = hipStreamWaitEvent(st, joined[i], 0);
    if (e != hipSuccess) return abandon_capture(e);
  }
  HIPC(launch_tick(d_clock, (uint64_t)graph_chunk, st));
  HIPC(hipStreamEndCapture(st, &graph[parts - 1]));
  HIPC(hipGraphInstantiate(&graph_exec[parts - 1], graph[parts - 1], nullptr, nullptr, 0));
  return FLB_OK;
}

int Group::step(uint64_t nsteps) {
  const int n = (int)P.size();
  const uint64_t K = (uint64_t)graph_chunk;
  const bool use_graph = graph_friendly();
  uint64_t done = 0;
  if (nsteps) at_work.begin(device);
  while (done < nsteps) {
    const uint64_t left = nsteps - done;
    if (use_graph && left >= K && t % K == 0 && steps_to_close(t, 0) >= K) {
      const bool others = at_work.others(device);
      const int parts = graph_branches(!others && !shared);
      shared = others;
      int rc = capture_graph(parts);
      if (rc != FLB_OK) return rc;
      hipGraphExec_t exec = graph_exec[parts - 1];
      if (profiling) {
        std::pair<hipEvent_t, hipEvent_t> ev;
        HIPC(hipEventCreate(&ev.first));
        HIPC(hipEventCreate(&ev.second));
        HIPC(hipEventRecord(ev.first, st));
        HIPC(hipGraphLaunch(exec, st));
        HIPC(hipEventRecord(ev.second, st));
        events.push_back(ev);
        prof_launches += K;
      } else {
        HIPC(hipGraphLaunch(exec, st));
      }
      for (uint64_t k = 0; k < K; ++k) {
        rc = after_step(t + k, true);
        if (rc != FLB_OK) return rc;
      }
      passed += graph_passed[parts - 1];
      t += K;
      done += K;
      continue;
    }
    // eager chunk: up to 2^30 steps; with graphs, only up to the next
    // multiple of the chunk length or the next time-block close, after which
    // replays can resume
    uint64_t chunk = std::min<uint64_t>(left, 1ull << 30);
    if (use_graph) {
      const uint64_t to_align = t % K == 0 ? K : K - t % K;
      chunk = std::min(chunk, std::min(to_align, std::max<uint64_t>(1, steps_to_close(t, 0))));
    }
    for (uint64_t k = 0; k < chunk; ++k) {
      const uint64_t tt = t + k;
      int pass[2];
      pass_pair(tt, chunk - k, true, &pass[0], &pass[1]);
      if (pass[1]) {
        for (int i = 0; i < 2; ++i) {
          int rc = profiled([&] { return launch_pass((uint32_t)k, t + k, pass[i], i); },
                            (uint64_t)pass[i]);
          for (int j = 0; j < pass[i] && rc == FLB_OK; ++j) rc = after_step(t + k + (uint64_t)j);
          if (rc != FLB_OK) return rc;
          k += (uint64_t)pass[i];
          passed += (uint64_t)pass[i];
        }
        --k;  // the loop's own step
        continue;
      }
      bool sample = false;
      for (int s = 0; s < n; ++s) sample |= sample_due(s, tt) || sk_due(s, tt);
      int rc = profiled(
          [&] { return launch_classes((uint32_t)k, sample, (int)(tt & 1), launch); }, 1);
      if (rc != FLB_OK) return rc;
      rc = after_step(tt);
      if (rc != FLB_OK) return rc;
    }
    HIPC(launch_tick(d_clock, chunk, st));
    t += chunk;
    done += chunk;
  }
  return FLB_OK;
}

hipError_t Group::wait() {
  const hipError_t e = hipStreamSynchronize(st);
  at_work.end();
  return e;
}

int Group::sync() {
  // waits for the stream too
  return read_errors(nullptr, 0);
}

// The error flags of every slot and the given pieces, in one readout behind
// the work enqueued so far; an error goes before the data.
int Group::read_errors(const HostPiece* more, int nmore) {
  const int n = (int)P.size();
  std::vector<int> err(n);
  std::vector<unsigned long long> es(n);
  std::vector<HostPiece> all{{err.data(), d_err, n * sizeof(int)},
                             {es.data(), d_err_step, n * sizeof(unsigned long long)}};
  all.insert(all.end(), more, more + nmore);
  HIPC(copy_out(all.data(), (int)all.size(), st, at_work.begun()));
  at_work.end();
  for (int s = 0; s < n; ++s) {
    err_step_host = -1;
    if (err[s]) {
      // own time of slot s at the failing step
      const int64_t stp = (int64_t)es[s];
      int code;
      if (err[s] & kErrInvalidVelocity) {
        code = set_error(FLB_E_INVALID_VELOCITY,
                         "lattice %d: local velocity outside the validity region at step %lld",
                         s, (long long)stp);
      } else {
        code = set_error(FLB_E_NONFINITE, "lattice %d: non-finite state at step %lld", s,
                         (long long)stp);
      }
      err_step_host = stp;
      return code;
    }
  }
  return FLB_OK;
}

// Nine planes of `rows` rows in d_io to rows r0 .. of host planes of N values.
int Group::copy_planes(void* dst, size_t N, size_t off, size_t B, size_t es) {
  if (B == N) {  // the whole lattice: one piece
    HIPC(copy_out(dst, d_io, 9 * N * es, st));
    return FLB_OK;
  }
  HostPiece p[9];
  for (int i = 0; i < 9; ++i)
    p[i] = {(char*)dst + (i * N + off) * es, (const char*)d_io + i * B * es, B * es};
  HIPC(copy_out(p, 9, st));
  return FLB_OK;
}

// The other way (synchronous for pageable memory).
int Group::copy_planes_in(const void* src, size_t N, size_t off, size_t B, size_t es) {
  if (B == N) {
    HIPC(hipMemcpyAsync(d_io, src, 9 * N * es, hipMemcpyHostToDevice, st));
    return FLB_OK;
  }
  for (int i = 0; i < 9; ++i)
    HIPC(hipMemcpyAsync((char*)d_io + i * B * es, (const char*)src + (i * N + off) * es, B * es,
                        hipMemcpyHostToDevice, st));
  return FLB_OK;
}

int Group::read_populations(int s, double* f) {
  return read_rows(s, 0, P[s].ny, f);
}

// Rows [y0, y0 + nrows) of slot s, unshifted FP64, [9][nrows][nx].
int Group::read_rows(int s, int y0, int nrows, double* f) {
  int rc = sync();
  if (rc != FLB_OK) return rc;
  const flb_params& p = P[s];
  if (y0 < 0 || nrows < 0 || y0 + nrows > p.ny)
    return set_error(FLB_E_ARG, "rows [%d, %d) outside 0..%d", y0, y0 + nrows, p.ny);
  const size_t N = (size_t)p.nx * nrows;
  for (int b0 = y0; b0 < y0 + nrows; b0 += band_rows) {
    const int rows = std::min(band_rows, y0 + nrows - b0);
    HIPC(launch_read_state(storage, pop[s], hdesc[s].pitch, d_io, p.nx, p.ny, (int)(t & 1), slot_shift(hdesc[s]),
                           b0, rows, st));
    rc = copy_planes(f, N, (size_t)(b0 - y0) * p.nx, (size_t)rows * p.nx, sizeof(double));
    if (rc != FLB_OK) return rc;
  }
  return FLB_OK;
}

int Group::set_populations(int s, const double* f, uint64_t tnew) {
  HIPC(wait());
  const flb_params& p = P[s];
  const size_t N = (size_t)p.nx * p.ny;
  if (P.size() != 1) return set_error(FLB_E_STATE, "set_populations needs a single lattice");
  t = tnew;
  HIPC(hipMemcpyAsync(d_clock, &t, sizeof(uint64_t), hipMemcpyHostToDevice, st));
  for (int y0 = 0; y0 < p.ny; y0 += band_rows) {
    const int rows = std::min(band_rows, p.ny - y0);
    const int rc = copy_planes_in(f, N, (size_t)y0 * p.nx, (size_t)rows * p.nx, sizeof(double));
    if (rc != FLB_OK) return rc;
    HIPC(launch_write_state(storage, pop[s], hdesc[s].pitch, d_io, p.nx, p.ny, (int)(t & 1), slot_shift(hdesc[s]),
                            y0, rows, st));
    HIPC(wait());
  }
  return FLB_OK;
}

int Group::set_fields(int s, const double* rho, const double* ux, const double* uy) {
  HIPC(wait());
  const flb_params& p = P[s];
  for (int y0 = 0; y0 < p.ny; y0 += band_rows) {
    const int rows = std::min(band_rows, p.ny - y0);
    const size_t B = (size_t)rows * p.nx, off = (size_t)y0 * p.nx;
    HIPC(hipMemcpyAsync(d_io, rho + off, B * sizeof(double), hipMemcpyHostToDevice, st));
    HIPC(hipMemcpyAsync(d_io + B, ux + off, B * sizeof(double), hipMemcpyHostToDevice, st));
    HIPC(hipMemcpyAsync(d_io + 2 * B, uy + off, B * sizeof(double), hipMemcpyHostToDevice, st));
    HIPC(launch_init(storage, pop[s], hdesc[s].pitch, d_io, d_io + B, d_io + 2 * B, p.rho0, p.ux0, p.uy0,
                     slot_shift(hdesc[s]), p.nx, p.ny, 0.0, hdesc[s].k0, hdesc[s].k1,
                     (int)(t & 1), y0, rows, st));
    HIPC(wait());
  }
  return FLB_OK;
}

int Group::read_moments(int s, int at, double* m) {
  int rc = sync();
  if (rc != FLB_OK) return rc;
  const flb_params& p = P[s];
  const size_t N = (size_t)p.nx * p.ny;
  const double* B = nullptr;
  if (at == FLB_AT_U0 || at == FLB_AT_HERMITE) {
    double h[81];
    if (at == FLB_AT_U0) std::memcpy(h, mt0[s].data(), sizeof(h));
    else hermite_rows(h);
    HIPC(hipMemcpyAsync(d_B, h, sizeof(h), hipMemcpyHostToDevice, st));
    HIPC(wait());
    B = d_B;
  } else if (at != FLB_AT_LOCAL) {
    return set_error(FLB_E_ARG, "unknown moment basis %d", at);
  }
  for (int y0 = 0; y0 < p.ny; y0 += band_rows) {
    const int rows = std::min(band_rows, p.ny - y0);
    HIPC(launch_moments(storage, pop[s], hdesc[s].pitch, B, d_io, p.nx, p.ny, (int)(t & 1), p.rho0, p.ux0,
                        p.uy0, slot_shift(hdesc[s]), d_err + s, y0, rows, st));
    rc = copy_planes(m, N, (size_t)y0 * p.nx, (size_t)rows * p.nx, sizeof(double));
    if (rc != FLB_OK) return rc;
  }
  return sync();
}

int Group::read_covariance(int s, flb_cov* out) {
  const flb_params& p = P[s];
  std::vector<double> rec;
  double open[kNStat] = {0};
  HostPiece piece[2];
  int n = 0;
  if (d_partials[s]) {
    HIPC(launch_open_sum(d_partials[s], hdesc[s].ntiles, d_open, d_open + kNStat, st));
    piece[n++] = {open, d_open, sizeof(open)};
    rec.resize((size_t)std::max<uint64_t>(stats[s].nb, 1) * kNStat);
    if (stats[s].nb > 0)
      piece[n++] = {rec.data(), d_records[s], stats[s].nb * kNStat * sizeof(double)};
  }
  const int rc = read_errors(piece, n);
  if (rc != FLB_OK) return rc;
  return finish_covariance(stats[s], rec, open, (uint64_t)p.nx * p.ny, mt0[s].data(), out);
}

int Group::reset_stats() {
  HIPC(wait());
  for (int s = 0; s < (int)P.size(); ++s) {
    stats[s].reset(P[s].block_steps);
    if (d_partials[s]) {
      HIPC(launch_fill(d_partials[s], (size_t)hdesc[s].ntiles * kNStat, 0.0, st));
      HIPC(launch_fill(d_records[s], (size_t)kMaxTimeBlocks * kNStat, 0.0, st));
    }
  }
  if (d_skacc) HIPC(launch_fill(d_skacc, 5 * sk_half(), 0.0, st));
  nsk = 0;
  HIPC(wait());
  return FLB_OK;
}

int Group::read_structure_factor(int which, double* out) {
  int rc = sync();
  if (rc != FLB_OK) return rc;
  if (!d_skacc) return set_error(FLB_E_STATE, "structure factors are off (sk_every = 0)");
  if (which < 0 || which > 4) return set_error(FLB_E_ARG, "unknown structure factor %d", which);
  const int nx = P[0].nx, ny = P[0].ny;
  const double norm = nsk > 0 ? 1.0 / ((double)nsk * (double)nx * (double)ny) : 0.0;
  // d_io holds 9 band_rows rows
  for (int k0 = 0; k0 < ny; k0 += 9 * band_rows) {
    const int rows = std::min(9 * band_rows, ny - k0);
    HIPC(launch_sk_expand(d_skacc + which * sk_half(), d_io, nx, ny, k0, rows, norm,
                          which == FLB_SK_JXJY_IM, st));
    HIPC(copy_out(out + (size_t)k0 * nx, d_io, (size_t)rows * nx * sizeof(double), st));
  }
  return FLB_OK;
}

int Group::read_fourier_mode(int which, int kx, int ky, double out[2]) {
  int rc = sync();
  if (rc != FLB_OK) return rc;
  if (which < 0 || which > 2) return set_error(FLB_E_ARG, "unknown field %d", which);
  const flb_params& p = P[0];
  const int nkx = ((kx % p.nx) + p.nx) % p.nx, nky = ((ky % p.ny) + p.ny) % p.ny;
  int gx, gy;
  const int nblocks = fourier_mode_grid(p.nx, p.ny, kModeBlocks, &gx, &gy);
  HIPC(launch_fourier_mode(storage, pop[0], hdesc[0].pitch, d_mode, kModeBlocks, p.nx, p.ny,
                           (int)(t & 1), which, nkx, nky, p.ux0, p.uy0, st));
  std::vector<double2> part(nblocks);
  HIPC(copy_out(part.data(), d_mode, nblocks * sizeof(double2), st));
  double sr = 0, si = 0;
  for (auto& v : part) {
    sr += v.x;
    si += v.y;
  }
  out[0] = sr;
  out[1] = si;
  return FLB_OK;
}

// Checkpoint layout: header, then the nine storage planes in natural order.
struct CkptHeader {
  char magic[8];
  uint64_t t;
  flb_params p;
  uint64_t payload;
};

size_t Group::checkpoint_bytes() const {
  return sizeof(CkptHeader) + 9 * (size_t)P[0].nx * P[0].ny * storage_size(storage);
}

int Group::checkpoint(void* host, size_t bytes) {
  int rc = sync();
  if (rc != FLB_OK) return rc;
  if (bytes < checkpoint_bytes()) return set_error(FLB_E_ARG, "checkpoint buffer too small");
  CkptHeader h;
  std::memset(&h, 0, sizeof(h));
  std::memcpy(h.magic, "FLBCKPT1", 8);
  h.t = t;
  h.p = P[0];
  h.payload = checkpoint_bytes() - sizeof(CkptHeader);
  std::memcpy(host, &h, sizeof(h));
  char* dst = (char*)host + sizeof(h);
  const flb_params& p = P[0];
  const size_t N = (size_t)p.nx * p.ny, es = storage_size(storage);
  for (int y0 = 0; y0 < p.ny; y0 += band_rows) {
    const int rows = std::min(band_rows, p.ny - y0);
    HIPC(launch_raw_state(storage, pop[0], hdesc[0].pitch, d_io, p.nx, p.ny, (int)(t & 1), 1, y0, rows, st));
    rc = copy_planes(dst, N, (size_t)y0 * p.nx, (size_t)rows * p.nx, es);
    if (rc != FLB_OK) return rc;
  }
  return FLB_OK;
}

int Group::restore(const void* host, size_t bytes) {
  HIPC(wait());
  if (bytes < sizeof(CkptHeader)) return set_error(FLB_E_ARG, "checkpoint too short");
  CkptHeader h;
  std::memcpy(&h, host, sizeof(h));
  if (std::memcmp(h.magic, "FLBCKPT1", 8) != 0) return set_error(FLB_E_ARG, "not a checkpoint");
  const flb_params& p = P[0];
  if (h.p.nx != p.nx || h.p.ny != p.ny || h.p.precision != p.precision ||
      h.payload + sizeof(h) != checkpoint_bytes() || bytes < checkpoint_bytes())
    return set_error(FLB_E_ARG, "checkpoint does not match this lattice");
  // the stored values are offsets from f^0(rho0, u0): the reference state must agree
  if (h.p.rho0 != p.rho0 || h.p.ux0 != p.ux0 || h.p.uy0 != p.uy0)
    return set_error(FLB_E_ARG, "checkpoint taken with another rho0 or u0");
  t = h.t;
  HIPC(hipMemcpyAsync(d_clock, &t, sizeof(uint64_t), hipMemcpyHostToDevice, st));
  const char* src = (const char*)host + sizeof(h);
  const size_t N = (size_t)p.nx * p.ny, es = storage_size(storage);
  for (int y0 = 0; y0 < p.ny; y0 += band_rows) {
    const int rows = std::min(band_rows, p.ny - y0);
    const int rc = copy_planes_in(src, N, (size_t)y0 * p.nx, (size_t)rows * p.nx, es);
    if (rc != FLB_OK) return rc;
    HIPC(launch_raw_state(storage, pop[0], hdesc[0].pitch, d_io, p.nx, p.ny, (int)(t & 1), 0, y0, rows, st));
    HIPC(wait());
  }
  return reset_stats();
}

int Group::kernel_time(double* ms, uint64_t* launches) {
  HIPC(wait());
  double tot = 0;
  for (auto& e : events) {
    float m = 0;
    HIPC(hipEventElapsedTime(&m, e.first, e.second));
    tot += m;
    (void)hipEventDestroy(e.first);
    (void)hipEventDestroy(e.second);
  }
  events.clear();
  prof_ms += tot;
  if (ms) *ms = prof_ms;
  if (launches) *launches = prof_launches;
  prof_ms = 0;
  prof_launches = 0;
  return FLB_OK;
}

}  // namespace flb

// ===================================================================== C ABI
using flb::Group;

struct flb_lattice {
  Group g;
};
struct flb_ensemble {
  Group g;
};

extern "C" {

const char* flb_last_error(void);

size_t flb_lattice_bytes(const flb_params* p) {
  if (flb::check_params(p) != FLB_OK) return 0;
  Group g;
  g.P.assign(p, p + 1);
  g.storage = p->precision == FLB_FP64 ? 0 : 1;
  g.hdesc.assign(1, flb::SlotDesc{});
  flb::fill_slot(p, &g.hdesc[0]);
  flb::Arena a;
  g.layout(a);
  return a.used + 256;
}

static int lattice_make(const flb_params* p, void* stream, void* buf, size_t bytes,
                        flb_lattice** out) {
  if (!out) return flb::set_error(FLB_E_ARG, "null output handle");
  *out = nullptr;
  flb_lattice* L = new (std::nothrow) flb_lattice();
  if (!L) return flb::set_error(FLB_E_OOM, "host allocation");
  const int rc = L->g.init(p, 1, stream, buf, bytes);
  if (rc != FLB_OK) {
    delete L;
    return rc;
  }
  *out = L;
  return FLB_OK;
}

int flb_lattice_create(const flb_params* p, void* hip_stream, flb_lattice** out) {
  return lattice_make(p, hip_stream, nullptr, 0, out);
}

int flb_lattice_create_on(const flb_params* p, void* dev_buf, size_t bytes, void* hip_stream,
                          flb_lattice** out) {
  if (!dev_buf) return flb::set_error(FLB_E_ARG, "null device buffer");
  return lattice_make(p, hip_stream, dev_buf, bytes, out);
}

#define NEED(h) \
  if (!(h)) return flb::set_error(FLB_E_ARG, "null handle")

int flb_lattice_set_fields(flb_lattice* L, const double* rho, const double* ux, const double* uy) {
  NEED(L);
  if (!rho || !ux || !uy) return flb::set_error(FLB_E_ARG, "null field");
  return L->g.set_fields(0, rho, ux, uy);
}
int flb_lattice_set_populations(flb_lattice* L, const double* f, uint64_t t) {
  NEED(L);
  if (!f) return flb::set_error(FLB_E_ARG, "null populations");
  return L->g.set_populations(0, f, t);
}
int flb_lattice_set_graph_chunk(flb_lattice* L, int32_t steps) {
  NEED(L);
  if (steps < 0 || steps > (1 << 16)) return flb::set_error(FLB_E_ARG, "bad chunk %d", steps);
  const hipError_t e = L->g.wait();  // no replay in flight
  if (e != hipSuccess) return flb::hip_fail(e, "sync");
  L->g.drop_graph();
  L->g.graph_chunk = steps + (steps & 1);  // even: replays keep the streaming phase
  return FLB_OK;
}
int flb_lattice_step(flb_lattice* L, uint64_t n) {
  NEED(L);
  return L->g.step(n);
}
int flb_lattice_sync(flb_lattice* L) {
  NEED(L);
  return L->g.sync();
}
int flb_lattice_read_populations(flb_lattice* L, double* f) {
  NEED(L);
  if (!f) return flb::set_error(FLB_E_ARG, "null output");
  return L->g.read_populations(0, f);
}
int flb_lattice_read_rows(flb_lattice* L, int32_t y0, int32_t nrows, double* f) {
  NEED(L);
  if (!f) return flb::set_error(FLB_E_ARG, "null output");
  return L->g.read_rows(0, y0, nrows, f);
}
int flb_lattice_read_moments(flb_lattice* L, int32_t at, double* m) {
  NEED(L);
  if (!m) return flb::set_error(FLB_E_ARG, "null output");
  return L->g.read_moments(0, at, m);
}
int flb_lattice_read_covariance(flb_lattice* L, flb_cov* out) {
  NEED(L);
  if (!out) return flb::set_error(FLB_E_ARG, "null output");
  return L->g.read_covariance(0, out);
}
int flb_lattice_read_structure_factor(flb_lattice* L, int32_t which, double* out) {
  NEED(L);
  if (!out) return flb::set_error(FLB_E_ARG, "null output");
  return L->g.read_structure_factor(which, out);
}
int flb_lattice_read_fourier_mode(flb_lattice* L, int32_t which, int32_t kx, int32_t ky,
                                  double out[2]) {
  NEED(L);
  if (!out) return flb::set_error(FLB_E_ARG, "null output");
  return L->g.read_fourier_mode(which, kx, ky, out);
}
int flb_lattice_reset_stats(flb_lattice* L) {
  NEED(L);
  return L->g.reset_stats();
}
size_t flb_lattice_checkpoint_bytes(flb_lattice* L) { return L ? L->g.checkpoint_bytes() : 0; }
int flb_lattice_checkpoint(flb_lattice* L, void* host, size_t bytes) {
  NEED(L);
  if (!host) return flb::set_error(FLB_E_ARG, "null buffer");
  return L->g.checkpoint(host, bytes);
}
int flb_lattice_restore(flb_lattice* L, const void* host, size_t bytes) {
  NEED(L);
  if (!host) return flb::set_error(FLB_E_ARG, "null buffer");
  return L->g.restore(host, bytes);
}
int flb_lattice_population_buffer(flb_lattice* L, void** dev, size_t* bytes, uint64_t* t) {
  NEED(L);
  if (!dev || !bytes || !t) return flb::set_error(FLB_E_ARG, "null output");
  const hipError_t e = L->g.wait();
  if (e != hipSuccess) return flb::hip_fail(e, "sync");
  const flb_params& p = L->g.P[0];
  *dev = L->g.pop[0];
  *bytes = flb::population_elems(p.nx, p.ny) * (L->g.storage == 0 ? 8 : 4);
  *t = L->g.t;
  return FLB_OK;
}
uint64_t flb_lattice_time(flb_lattice* L) { return L ? L->g.t : 0; }
int64_t flb_lattice_error_step(flb_lattice* L) { return L ? L->g.err_step_host : -1; }
int flb_lattice_profile(flb_lattice* L, int32_t on) {
  NEED(L);
  L->g.profiling = on != 0;
  return FLB_OK;
}
int flb_lattice_kernel_time(flb_lattice* L, double* ms, uint64_t* launches) {
  NEED(L);
  return L->g.kernel_time(ms, launches);
}
int flb_lattice_pass_steps(flb_lattice* L, uint64_t* steps) {
  NEED(L);
  if (!steps) return flb::set_error(FLB_E_ARG, "null output");
  *steps = L->g.passed;
  return FLB_OK;
}
void flb_lattice_destroy(flb_lattice* L) { delete L; }

int flb_ensemble_create(const flb_params* ps, int32_t n, void* hip_stream, flb_ensemble** out) {
  if (!out || !ps) return flb::set_error(FLB_E_ARG, "null argument");
  *out = nullptr;
  flb_ensemble* E = new (std::nothrow) flb_ensemble();
  if (!E) return flb::set_error(FLB_E_OOM, "host allocation");
  const int rc = E->g.init(ps, n, hip_stream, nullptr, 0);
  if (rc != FLB_OK) {
    delete E;
    return rc;
  }
  *out = E;
  return FLB_OK;
}
int flb_ensemble_set_graph_chunk(flb_ensemble* E, int32_t steps) {
  NEED(E);
  if (steps < 0 || steps > (1 << 16)) return flb::set_error(FLB_E_ARG, "bad chunk %d", steps);
  const hipError_t e = E->g.wait();  // no replay in flight
  if (e != hipSuccess) return flb::hip_fail(e, "sync");
  E->g.drop_graph();
  E->g.graph_chunk = steps + (steps & 1);  // even: replays keep the streaming phase
  return FLB_OK;
}
int flb_ensemble_step(flb_ensemble* E, uint64_t n) {
  NEED(E);
  return E->g.step(n);
}
int flb_ensemble_sync(flb_ensemble* E) {
  NEED(E);
  return E->g.sync();
}
int flb_ensemble_read_populations(flb_ensemble* E, int32_t i, double* f) {
  NEED(E);
  if (i < 0 || i >= (int)E->g.P.size() || !f) return flb::set_error(FLB_E_ARG, "bad replica");
  return E->g.read_populations(i, f);
}
int flb_ensemble_read_covariance(flb_ensemble* E, int32_t i, flb_cov* out) {
  NEED(E);
  if (i < 0 || i >= (int)E->g.P.size() || !out) return flb::set_error(FLB_E_ARG, "bad replica");
  return E->g.read_covariance(i, out);
}
int flb_ensemble_reset_stats(flb_ensemble* E) {
  NEED(E);
  return E->g.reset_stats();
}
uint64_t flb_ensemble_time(flb_ensemble* E) { return E ? E->g.t : 0; }
int flb_ensemble_profile(flb_ensemble* E, int32_t on) {
  NEED(E);
  E->g.profiling = on != 0;
  return FLB_OK;
}
int flb_ensemble_kernel_time(flb_ensemble* E, double* ms, uint64_t* launches) {
  NEED(E);
  return E->g.kernel_time(ms, launches);
}
int flb_ensemble_pass_steps(flb_ensemble* E, uint64_t* steps) {
  NEED(E);
  if (!steps) return flb::set_error(FLB_E_ARG, "null output");
  *steps = E->g.passed;
  return FLB_OK;
}
void flb_ensemble_destroy(flb_ensemble* E) { delete E; }

int flb_lattice_autotune(flb_lattice* L, int32_t reps, flb_launch_config* results,
                         int32_t max_results, int32_t* n_results) {
  NEED(L);
  return L->g.autotune(reps, results, max_results, n_results);
}
int flb_ensemble_autotune(flb_ensemble* E, int32_t reps, flb_launch_config* results,
                          int32_t max_results, int32_t* n_results) {
  NEED(E);
  return E->g.autotune(reps, results, max_results, n_results);
}
int flb_lattice_set_launch(flb_lattice* L, const flb_launch_config* c) {
  NEED(L);
  return L->g.set_launch(c);
}
int flb_ensemble_set_launch(flb_ensemble* E, const flb_launch_config* c) {
  NEED(E);
  return E->g.set_launch(c);
}
int flb_lattice_get_launch(flb_lattice* L, flb_launch_config* c) {
  NEED(L);
  if (!c) return flb::set_error(FLB_E_ARG, "null output");
  *c = flb_launch_config{L->g.launch.tiles_per_block, L->g.launch.grid_blocks, 0.0};
  return FLB_OK;
}
int flb_ensemble_get_launch(flb_ensemble* E, flb_launch_config* c) {
  NEED(E);
  if (!c) return flb::set_error(FLB_E_ARG, "null output");
  *c = flb_launch_config{E->g.launch.tiles_per_block, E->g.launch.grid_blocks, 0.0};
  return FLB_OK;
}

}  // extern "C"
