// flb_server.cpp — continuous batching of simulation requests.
//
// Requests wait in arrival order.  At every chunk boundary the scheduler
// retires finished requests (their correlators are read and their memory
// returned), then admits waiting requests in order while a slot is free and
// the head request's device footprint fits the memory budget (a first-fit
// arena carved from one allocation of the budget).  All admitted requests
// then advance together for `chunk_steps` steps: one batched step launch
// per step and compute precision, or one for each of two halves on two streams,
// covers every active lattice; a request that
// reaches its step count stops updating inside the chunk.  A request runs
// on its own clock (t = t0 + device clock), with noise keyed by its own
// seed, step and site and its correlator sums reduced per request in a
// fixed order, so its result does not depend on what else is in the batch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <condition_variable>
#include <cstring>
#include <deque>
#include <map>
#include <mutex>
#include <thread>
#include <vector>

#include "flb.h"
#include "flb_runtime.hpp"

namespace flb {

constexpr int kServerBlocks = 64;  // time-block records per request

#define HIPC(expr)                                    \
  do {                                                \
    hipError_t e_ = (expr);                           \
    if (e_ != hipSuccess) return hip_fail(e_, #expr); \
  } while (0)

// First-fit allocator over [0, cap).
struct FreeList {
  std::map<size_t, size_t> free;  // offset -> size
  size_t cap = 0, used = 0;
  void reset(size_t c) {
    cap = c;
    used = 0;
    free.clear();
    free[0] = c;
  }
  bool alloc(size_t n, size_t* off) {
    n = (n + 255) & ~(size_t)255;
    for (auto it = free.begin(); it != free.end(); ++it) {
      if (it->second >= n) {
        *off = it->first;
        const size_t rest = it->second - n, o = it->first + n;
        free.erase(it);
        if (rest) free[o] = rest;
        used += n;
        return true;
      }
    }
    return false;
  }
  void release(size_t off, size_t n) {
    n = (n + 255) & ~(size_t)255;
    used -= n;
    auto it = free.emplace(off, n).first;
    auto nx = std::next(it);
    if (nx != free.end() && it->first + it->second == nx->first) {
      it->second += nx->second;
      free.erase(nx);
    }
    if (it != free.begin()) {
      auto pv = std::prev(it);
      if (pv->first + pv->second == it->first) {
        pv->second += it->second;
        free.erase(it);
      }
    }
  }
};

struct Request {
  uint64_t id;
  flb_request r;
  double t_submit;
};

struct Active {
  uint64_t id, tag, nsteps;
  flb_params p;
  double t_submit, t_admit;
  size_t off = 0, bytes = 0;
  SlotDesc desc;
  Stats stats;
  int cls = 1;  // compute class: 0 FP64, 1 FP32
};

static size_t request_bytes_of(const flb_params& p, int storage) {
  int wide = 0, tiles_x = 0, ntiles = 0;
  tile_shape(p, &wide, &tiles_x, &ntiles);
  size_t b = population_elems(p.nx, p.ny) * (storage == 0 ? 8 : 4);
  b = (b + 255) & ~(size_t)255;
  if (p.sample_every > 0) {
    b += ((size_t)ntiles * kNStat * 8 + 255) & ~(size_t)255;
    b += ((size_t)kServerBlocks * kNStat * 8 + 255) & ~(size_t)255;
  }
  b += 256;  // error flag and step
  return b;
}

}  // namespace flb

using namespace flb;

struct flb_server {
  Staging staging;
  flb_server_config cfg;
  hipStream_t st = nullptr;
  bool own_stream = false;
  char *arena = nullptr, *tables = nullptr;
  FreeList fl;
  std::mutex mu;
  std::condition_variable cv, done_cv;
  std::deque<Request> queue;
  std::deque<flb_result> results;
  std::vector<Active> active;
  uint64_t next_id = 1, submitted = 0, completed = 0;
  uint64_t clock = 0;  // server steps so far (mirrors the device clock)
  // device tables per compute class
  SlotDesc* d_slots[2] = {nullptr, nullptr};
  int* d_prefix[2] = {nullptr, nullptr};
  uint64_t* d_clock = nullptr;
  double* d_open = nullptr;
  std::vector<SlotDesc> h_slots[2];
  std::vector<int> h_prefix[2];
  // the second of the two streams a chunk may run on, and the events that
  // fork and join it
  hipStream_t st2 = nullptr;
  hipEvent_t forked = nullptr, joined = nullptr;
  int device = 0;
  AtWork at_work;
  std::chrono::steady_clock::time_point t_start;
  double busy = 0;
  std::thread worker;
  bool stop = false;
  int error = FLB_OK;

  double now() const {
    return std::chrono::duration<double>(std::chrono::steady_clock::now() - t_start).count();
  }
  int admit_locked();
  int finish(const Active& a);
  int retire();
  int run_chunk();
  int pump(int max_chunks, int* did);
};

int flb_server::admit_locked() {
  while (!queue.empty() && (int)active.size() < cfg.max_slots) {
    Request& q = queue.front();
    const size_t bytes = request_bytes_of(q.r.p, cfg.precision);
    size_t off = 0;
    if (!fl.alloc(bytes, &off)) break;  // head waits for memory (FIFO)
    Active a;
    a.id = q.id;
    a.tag = q.r.tag;
    a.nsteps = q.r.nsteps;
    a.p = q.r.p;
    a.t_submit = q.t_submit;
    a.t_admit = now();
    a.off = off;
    a.bytes = bytes;
    std::memset(&a.desc, 0, sizeof(a.desc));
    fill_slot(&a.p, &a.desc);
    a.cls = compute_precision(&a.p);
    char* base = arena + off;
    size_t o = 0;
    auto take = [&](size_t n) {
      char* p = base + o;
      o += (n + 255) & ~(size_t)255;
      return p;
    };
    a.desc.pop = take(population_elems(a.p.nx, a.p.ny) * (cfg.precision == 0 ? 8 : 4));
    if (a.p.sample_every > 0) {
      a.desc.partials = (double*)take((size_t)a.desc.ntiles * kNStat * 8);
      a.stats.max_blocks = kServerBlocks;
    }
    double* records = a.p.sample_every > 0 ? (double*)take((size_t)kServerBlocks * kNStat * 8)
                                           : nullptr;
    a.desc.err = (int*)take(8);
    a.desc.err_step = (unsigned long long*)(a.desc.err + 2);
    a.desc.skz = nullptr;
    a.desc.t0 = (uint64_t)0 - clock;  // own time 0 at the current server clock
    a.desc.tend = a.nsteps;
    a.stats.reset(a.p.block_steps);
    // state: equilibrium (or thermal) start, cleared sums and flags
    const double mu = a.p.init == FLB_INIT_THERMAL ? 3.0 * a.p.kT : 0.0;
    hipError_t e = launch_init(cfg.precision == 0 ? 0 : 1, a.desc.pop, a.desc.pitch, nullptr,
                               nullptr, nullptr, a.p.rho0, a.p.ux0, a.p.uy0, slot_shift(a.desc), a.p.nx, a.p.ny,
                               mu, a.desc.k0, a.desc.k1, 0, 0, a.p.ny, st);
    if (e == hipSuccess && a.desc.partials) {
      e = launch_fill(a.desc.partials, (size_t)a.desc.ntiles * kNStat, 0.0, st);
      if (e == hipSuccess) e = launch_fill(records, (size_t)kServerBlocks * kNStat, 0.0, st);
    }
    if (e == hipSuccess) e = hipMemsetAsync(a.desc.err, 0, 4, st);
    if (e == hipSuccess) e = hipMemsetAsync(a.desc.err_step, 0xFF, 8, st);
    if (e != hipSuccess) {
      fl.release(off, bytes);  // the request stays queued
      return hip_fail(e, "request set-up");
    }
    active.push_back(a);
    queue.pop_front();
  }
  return FLB_OK;
}

static double* records_of(const Active& a, char* arena, int precision) {
  if (a.p.sample_every <= 0) return nullptr;
  size_t o = (population_elems(a.p.nx, a.p.ny) * (precision == 0 ? 8 : 4) + 255) & ~(size_t)255;
  o += ((size_t)a.desc.ntiles * kNStat * 8 + 255) & ~(size_t)255;
  return (double*)(arena + a.off + o);
}

// Reads the correlators of a request that reached its step count, queues its
// result and returns its memory.  On a HIP error nothing is released.
int flb_server::finish(const Active& a) {
  flb_result res;
  std::memset(&res, 0, sizeof(res));
  res.id = a.id;
  res.tag = a.tag;
  res.nsteps = a.nsteps;
  res.t_submit = a.t_submit;
  res.t_admit = a.t_admit;
  int err = 0;
  double open[kNStat];
  std::vector<double> recs((size_t)std::max<uint64_t>(a.stats.nb, 1) * kNStat);
  HostPiece piece[3] = {{&err, a.desc.err, 4}};
  int n = 1;
  if (a.desc.partials) {
    HIPC(launch_open_sum(a.desc.partials, a.desc.ntiles, d_open, d_open + kNStat, st));
    piece[n++] = {open, d_open, sizeof(open)};
    if (a.stats.nb)
      piece[n++] = {recs.data(), records_of(a, arena, cfg.precision), a.stats.nb * kNStat * 8};
  }
  HIPC(copy_out(piece, n, st));
  res.status = err ? ((err & kErrInvalidVelocity) ? FLB_E_INVALID_VELOCITY : FLB_E_NONFINITE)
                   : FLB_OK;
  if (a.desc.partials && !err) {
    double mt0[81];
    fnorm_rows(a.p.ux0, a.p.uy0, mt0);
    finish_covariance(a.stats, recs, open, (uint64_t)a.p.nx * a.p.ny, mt0, &res.cov);
  }
  res.t_done = now();
  fl.release(a.off, a.bytes);
  {
    std::lock_guard<std::mutex> lk(mu);
    results.push_back(res);
    completed += 1;
  }
  done_cv.notify_all();
  return FLB_OK;
}

// Retires every request whose own time reached nsteps.  The list of active
// requests is replaced under the lock (other threads read its size); after a
// failure the requests not yet retired stay in it.
int flb_server::retire() {
  HIPC(hipStreamSynchronize(st));
  at_work.end();
  std::vector<Active> keep;
  int rc = FLB_OK;
  for (const Active& a : active) {
    if (rc == FLB_OK && a.desc.t0 + clock >= a.nsteps) {
      rc = finish(a);
      if (rc == FLB_OK) continue;
    }
    keep.push_back(a);
  }
  std::lock_guard<std::mutex> lk(mu);
  active.swap(keep);
  return rc;
}

// One chunk: upload the slot tables, launch chunk_steps batched steps, tick.
// Requests do not depend on each other, so the requests of a class are dealt
// to two halves of about the same number of tiles that advance on two streams,
// one filling the chip while the other's step ends, where the steps are long
// enough for twice the launches (two_branches).
int flb_server::run_chunk() {
  const int K = cfg.chunk_steps;
  struct Half {
    int cls, first, count, tiles, prefix_at;
    hipStream_t q;
  };
  std::vector<Half> halves;
  std::vector<hipStream_t> stream_of(active.size(), st);
  bool two = false;
  at_work.begin(device);
  const bool alone = !at_work.others(device);
  for (int c = 0; c < 2; ++c) {
    h_slots[c].clear();
    h_prefix[c].clear();
    int total = 0, n = 0;
    for (auto& a : active)
      if (a.cls == c) {
        total += a.desc.ntiles;
        ++n;
      }
    if (!n) continue;
    const bool split = n > 1 && two_branches(c, total, alone);
    // in order, each request to the lighter half
    int load[2] = {0, 0};
    std::vector<int> half(active.size(), 0);
    if (split)
      for (size_t i = 0; i < active.size(); ++i)
        if (active[i].cls == c) {
          half[i] = load[1] < load[0];
          load[half[i]] += active[i].desc.ntiles;
        }
    for (int p = 0; p < (split ? 2 : 1); ++p) {
      Half h{c, (int)h_slots[c].size(), 0, 0, (int)h_prefix[c].size(), p ? st2 : st};
      h_prefix[c].push_back(0);
      for (size_t i = 0; i < active.size(); ++i) {
        if (active[i].cls != c || half[i] != p) continue;
        h_slots[c].push_back(active[i].desc);
        h.tiles += active[i].desc.ntiles;
        h_prefix[c].push_back(h.tiles);
        ++h.count;
        stream_of[i] = h.q;
      }
      if (h.count) halves.push_back(h);
      two = two || (p == 1 && h.count);
    }
    HIPC(hipMemcpyAsync(d_slots[c], h_slots[c].data(), h_slots[c].size() * sizeof(SlotDesc),
                        hipMemcpyHostToDevice, st));
    HIPC(hipMemcpyAsync(d_prefix[c], h_prefix[c].data(), h_prefix[c].size() * sizeof(int),
                        hipMemcpyHostToDevice, st));
  }
  if (two) {
    HIPC(hipEventRecord(forked, st));
    HIPC(hipStreamWaitEvent(st2, forked, 0));
  }
  const int storage = cfg.precision == 0 ? 0 : 1;
  // Time blocks that end at a step, the requests of a stream in one pair of
  // launches.  Twelve requests (sides 93 to 980, a block every 50 steps): 137
  // pairs of 15 us became 38 of 25, half of them beside the other stream's
  // steps; 27.4 -> 26.2 ms in all.
  std::vector<double*> partials[2], records[2];
  std::vector<int> ntiles[2];
  for (int k = 0; k < K; ++k) {
    for (const Half& h : halves) {
      // the sampling variant only where some request of the half samples
      bool due = false;
      for (int i = h.first; i < h.first + h.count; ++i) {
        const SlotDesc& d = h_slots[h.cls][i];
        const uint64_t own = d.t0 + clock + (uint64_t)k;
        due |= own < d.tend && d.sample_every > 0 && own % (uint64_t)d.sample_every == 0;
      }
      // chunk_steps is even, so every request's own time has the parity of k
      HIPC(launch_step(storage, h.cls, cfg.basis, due, k & 1, d_slots[h.cls] + h.first,
                       d_prefix[h.cls] + h.prefix_at, h.count, h.tiles, d_clock, (uint32_t)k,
                       LaunchCfg{}, h.q));
    }
    for (int q = 0; q < 2; ++q) {
      partials[q].clear();
      records[q].clear();
      ntiles[q].clear();
    }
    for (size_t i = 0; i < active.size(); ++i) {
      Active& a = active[i];
      const uint64_t own = a.desc.t0 + clock + (uint64_t)k;
      if (own >= a.nsteps || a.p.sample_every <= 0) continue;
      if (own % (uint64_t)a.p.sample_every != 0) continue;
      if (a.stats.plain_close_next()) {
        const int q = stream_of[i] == st2;
        const uint64_t b = a.stats.close_counted((uint64_t)a.p.nx * a.p.ny);
        partials[q].push_back(a.desc.partials);
        records[q].push_back(records_of(a, arena, cfg.precision) + b * kNStat);
        ntiles[q].push_back(a.desc.ntiles);
        continue;
      }
      HIPC(a.stats.after_sample((uint64_t)a.p.nx * a.p.ny, a.desc.partials, a.desc.ntiles,
                                records_of(a, arena, cfg.precision), stream_of[i]));
    }
    for (int q = 0; q < 2; ++q)
      if (!ntiles[q].empty())
        HIPC(launch_close_block_list(partials[q].data(), records[q].data(), ntiles[q].data(),
                                     (int)ntiles[q].size(), q ? st2 : st));
  }
  if (two) {
    HIPC(hipEventRecord(joined, st2));
    HIPC(hipStreamWaitEvent(st, joined, 0));
  }
  HIPC(launch_tick(d_clock, (uint64_t)K, st));
  clock += (uint64_t)K;
  return FLB_OK;
}

int flb_server::pump(int max_chunks, int* did) {
  int n = 0;
  for (; n < max_chunks; ++n) {
    {
      std::lock_guard<std::mutex> lk(mu);
      const int rc = admit_locked();
      if (rc != FLB_OK) return rc;
    }
    if (active.empty()) break;
    const double t0 = now();
    int rc = run_chunk();
    if (rc != FLB_OK) {
      // the next chunk's tables go to st alone: nothing of this one may still
      // run on the second stream
      (void)hipStreamSynchronize(st2);
      return rc;
    }
    rc = retire();
    if (rc != FLB_OK) return rc;
    std::lock_guard<std::mutex> lk(mu);
    busy += now() - t0;
  }
  if (did) *did = n;
  return FLB_OK;
}

extern "C" {

size_t flb_server_request_bytes(const flb_server_config* cfg, const flb_request* r) {
  if (!cfg || !r) return 0;
  flb_params p = r->p;
  p.precision = cfg->precision;
  p.basis = cfg->basis;
  if (flb::check_params(&p) != FLB_OK) return 0;
  return request_bytes_of(p, cfg->precision == FLB_FP64 ? 0 : 1);
}

int flb_server_create(const flb_server_config* cfg, void* hip_stream, flb_server** out) {
  if (!cfg || !out) return set_error(FLB_E_ARG, "null argument");
  *out = nullptr;
  if (cfg->max_slots <= 0 || cfg->chunk_steps <= 0 || cfg->mem_budget_bytes < 4096)
    return set_error(FLB_E_ARG, "bad server configuration");
  if (cfg->precision != FLB_FP64 && cfg->precision != FLB_FP32_SHIFTED)
    return set_error(FLB_E_ARG, "unknown precision");
  if (cfg->basis < 0 || cfg->basis > 2) return set_error(FLB_E_ARG, "unknown basis");
  flb_server* S = new (std::nothrow) flb_server();
  if (!S) return set_error(FLB_E_OOM, "host allocation");
  S->cfg = *cfg;
  S->cfg.chunk_steps += S->cfg.chunk_steps & 1;  // even: all requests share the streaming phase
  S->t_start = std::chrono::steady_clock::now();
  auto fail = [&](int rc) {
    flb_server_destroy(S);
    return rc;
  };
  hipError_t e = hipGetDevice(&S->device);
  if (e != hipSuccess) return fail(hip_fail(e, "device"));
  if (hip_stream) {
    S->st = (hipStream_t)hip_stream;
  } else {
    e = hipStreamCreateWithFlags(&S->st, hipStreamNonBlocking);
    if (e != hipSuccess) return fail(hip_fail(e, "stream"));
    S->own_stream = true;
  }
  e = hipStreamCreateWithFlags(&S->st2, hipStreamNonBlocking);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&S->forked, hipEventDisableTiming);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&S->joined, hipEventDisableTiming);
  if (e != hipSuccess) return fail(hip_fail(e, "second stream"));
  e = hipMalloc((void**)&S->arena, cfg->mem_budget_bytes);
  if (e != hipSuccess) return fail(set_error(FLB_E_OOM, "server arena of %zu bytes",
                                             cfg->mem_budget_bytes));
  S->fl.reset(cfg->mem_budget_bytes);
  // the slot tables, the clock and the open sums in one allocation
  for (int pass = 0; pass < 2; ++pass) {
    Arena a;
    a.base = S->tables;
    for (int c = 0; c < 2; ++c) {
      S->d_slots[c] = a.take<SlotDesc>(cfg->max_slots);
      S->d_prefix[c] = a.take<int>((size_t)cfg->max_slots + 2);  // of two halves
    }
    S->d_clock = a.take<uint64_t>(1);
    S->d_open = a.take<double>((size_t)(1 + kFoldRows) * kNStat);
    if (pass == 0 && hipMalloc((void**)&S->tables, a.used) != hipSuccess)
      return fail(set_error(FLB_E_OOM, "slot tables"));
  }
  e = hipMemsetAsync(S->d_clock, 0, 8, S->st);
  if (e == hipSuccess) e = hipStreamSynchronize(S->st);
  if (e != hipSuccess) return fail(hip_fail(e, "clock init"));
  if (cfg->threaded) {
    S->worker = std::thread([S] {
      while (true) {
        {
          std::unique_lock<std::mutex> lk(S->mu);
          S->cv.wait(lk, [S] { return S->stop || !S->queue.empty() || !S->active.empty(); });
          if (S->stop) return;
        }
        int did = 0;
        const int rc = S->pump(1, &did);
        if (rc != FLB_OK) {
          std::lock_guard<std::mutex> lk(S->mu);
          S->error = rc;
          S->stop = true;
          S->done_cv.notify_all();
          return;
        }
        if (did == 0) {
          // nothing admissible: wait for a new submission
          std::unique_lock<std::mutex> lk(S->mu);
          S->cv.wait_for(lk, std::chrono::milliseconds(1));
        }
      }
    });
  }
  *out = S;
  return FLB_OK;
}

int flb_server_submit(flb_server* S, const flb_request* r, uint64_t* id) {
  if (!S || !r) return set_error(FLB_E_ARG, "null argument");
  flb_request q = *r;
  q.p.precision = S->cfg.precision;
  q.p.basis = S->cfg.basis;
  q.p.sk_every = 0;
  int rc = check_params(&q.p);
  if (rc != FLB_OK) return rc;
  if (q.nsteps == 0) return set_error(FLB_E_ARG, "request needs at least one step");
  if (q.nsteps >= (1ull << 62)) return set_error(FLB_E_ARG, "request of 2^62 steps or more");
  if (request_bytes_of(q.p, S->cfg.precision) > S->cfg.mem_budget_bytes)
    return set_error(FLB_E_ADMISSION, "request footprint exceeds the memory budget");
  {
    std::lock_guard<std::mutex> lk(S->mu);
    if (S->stop) return set_error(FLB_E_ADMISSION, "server stopped (error %d)", S->error);
    Request rq;
    rq.id = S->next_id++;
    rq.r = q;
    rq.t_submit = S->now();
    S->queue.push_back(rq);
    S->submitted += 1;
    if (id) *id = rq.id;
  }
  S->cv.notify_all();
  return FLB_OK;
}

int flb_server_pump(flb_server* S, int32_t max_chunks, int32_t* did_work) {
  if (!S) return set_error(FLB_E_ARG, "null server");
  if (S->cfg.threaded) return set_error(FLB_E_STATE, "threaded server pumps itself");
  int did = 0;
  const int rc = S->pump(max_chunks, &did);
  if (did_work) *did_work = did;
  return rc;
}

int flb_server_poll(flb_server* S, flb_result* out, int32_t max, int32_t* n) {
  if (!S || !n || (max > 0 && !out)) return set_error(FLB_E_ARG, "null argument");
  std::lock_guard<std::mutex> lk(S->mu);
  int k = 0;
  while (k < max && !S->results.empty()) {
    out[k++] = S->results.front();
    S->results.pop_front();
  }
  *n = k;
  return S->error;
}

int flb_server_drain(flb_server* S) {
  if (!S) return set_error(FLB_E_ARG, "null server");
  if (!S->cfg.threaded) {
    while (true) {
      {
        std::lock_guard<std::mutex> lk(S->mu);
        if (S->completed == S->submitted) return FLB_OK;
      }
      int did = 0;
      const int rc = S->pump(1 << 20, &did);
      if (rc != FLB_OK) return rc;
      if (did == 0 && S->active.empty()) {
        std::lock_guard<std::mutex> lk(S->mu);
        if (!S->queue.empty()) return set_error(FLB_E_ADMISSION, "queued request cannot be admitted");
      }
    }
  }
  std::unique_lock<std::mutex> lk(S->mu);
  S->done_cv.wait(lk, [S] { return S->completed == S->submitted || S->stop; });
  return S->error;
}

int flb_server_stats(flb_server* S, int32_t* queued, int32_t* active, uint64_t* completed,
                     double* busy_seconds, double* wall_seconds) {
  if (!S) return set_error(FLB_E_ARG, "null server");
  std::lock_guard<std::mutex> lk(S->mu);
  if (queued) *queued = (int32_t)S->queue.size();
  if (active) *active = (int32_t)S->active.size();
  if (completed) *completed = S->completed;
  if (busy_seconds) *busy_seconds = S->busy;
  if (wall_seconds) *wall_seconds = S->now();
  return FLB_OK;
}

void flb_server_destroy(flb_server* S) {
  if (!S) return;
  {
    std::lock_guard<std::mutex> lk(S->mu);
    S->stop = true;
  }
  S->cv.notify_all();
  if (S->worker.joinable()) S->worker.join();
  if (S->st2) (void)hipStreamSynchronize(S->st2);
  if (S->st) (void)hipStreamSynchronize(S->st);
  if (S->tables) (void)hipFree(S->tables);
  if (S->arena) (void)hipFree(S->arena);
  if (S->forked) (void)hipEventDestroy(S->forked);
  if (S->joined) (void)hipEventDestroy(S->joined);
  if (S->st2) (void)hipStreamDestroy(S->st2);
  if (S->own_stream && S->st) (void)hipStreamDestroy(S->st);
  delete S;
}

}  // extern "C"
