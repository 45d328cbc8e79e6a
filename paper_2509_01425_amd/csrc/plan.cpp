// plan.cpp -- persistent memcpy batches replayed from a HIP graph.
//
// A plan is a batch of memcpy requests (HiCR Sec. 3.1.4) that a caller
// repeats unchanged.  Validation, address resolution, the upload, the split
// into copy launches and (for batches of more than 4,096 requests) the scan
// of the piece table happen once.  A replay queues the copy launches again,
// and is counted in the slot table (a plan that writes host memory: by a
// counter kernel), or is -- HICR_PLAN_GRAPH -- one hipGraphLaunch of copy
// launches and counter kernel captured from a private stream at creation.  The graph holds kernel nodes only; nothing in
// it needs clearing between replays.  (Measured on gfx950 with ROCm 7: a
// graph of two or five kernel nodes launches slower than the same kernels
// queued directly, so direct replay is the default.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <utility>
#include <vector>

#include "replays.h"
#include "runtime.h"

using namespace hicr;

struct hicr_plan_s {
  hicr_ctx c = nullptr;
  uint64_t n = 0;
  // device: kHead bytes of head (the arrival counter), the SoA {dst, src, size,
  // slot pair} (32 B per request), then the piece tables (8 B per request) or
  // the stream kernel's starts
  void *d = nullptr;
  uint64_t *batch() const { return d ? static_cast<uint64_t *>(d) + kHead / 8 : nullptr; }
  static constexpr size_t kHead = 128;
  std::vector<Seg> segs;      // copy launches of one replay
  uint32_t waves = 0;         // waves of the stream kernel (0: the piece kernels)
  const StreamStart *starts = nullptr;  // their shares
  // A stream plan's shares under each copy grid it has been launched with:
  // waves and starts.  Kept until the plan goes, as a replay in flight or a graph
  // of the caller's may read them; h: destinations and sizes, to cut more.
  int per_cu = 0;             // the copy grid of `waves` and `starts`
  std::map<int, std::pair<uint32_t, const StreamStart *>> cuts;
  std::vector<void *> more;   // device buffers of the cuts that came later
  std::vector<uint64_t> h;
  uint64_t bytes = 0, host_bytes = 0, n_short = 0;
  uint32_t share(int grid) const;  // its waves under a copy grid
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;  // HICR_PLAN_GRAPH
  DevSched ds{};
  Signal sig;                 // end of the last replay; seq counts the replays
  hipStream_t last = nullptr; // stream of the last replay
  bool launched = false;
  std::vector<hicr_slot> slots;  // distinct slots the requests name
  // direct replays of a plan that writes device memory only: their copy
  // launch raises sig's words, and a replay is counted in the slots here
  // (sent and received per entry of `slots`)
  bool host_count = false;
  Replays replays;
  std::vector<uint64_t> n_sent, n_recv;
};

uint32_t hicr_plan_s::share(int grid) const {
  return stream_waves(n, bytes, c->n_cu, grid, n_short, 2 * host_bytes > bytes);
}

namespace {

void free_plan(hicr_plan p) {
  if (p->exec) (void)hipGraphExecDestroy(p->exec);
  if (p->graph) (void)hipGraphDestroy(p->graph);
  if (p->sig.ev) (void)hipEventDestroy(p->sig.ev);
  if (p->d) (void)hipFree(p->d);
  for (void *d : p->more) (void)hipFree(d);
  if (p->sig.words) p->c->plan_words.push_back(p->sig.words);
  for (hicr_slot s : p->slots) p->c->slots[s].plan_refs--;
  delete p;
}

// Done words of a plan (pinned), from blocks the context keeps.
hipError_t take_words(hicr_ctx c, uint64_t **out) {
  if (c->plan_words.empty()) {
    constexpr int kPlans = 16;
    void *b = nullptr;
    hipError_t e = hipHostMalloc(&b, 8 * kDoneWords * kPlans, hipHostMallocDefault);
    if (e != hipSuccess) return e;
    c->plan_blocks.push_back(b);
    for (int i = 0; i < kPlans; i++)
      c->plan_words.push_back(static_cast<uint64_t *>(b) + kDoneWords * i);
  }
  *out = c->plan_words.back();
  c->plan_words.pop_back();
  std::memset(*out, 0, 8 * kDoneWords);
  return hipSuccess;
}

// The slots that requests name, each once, in ascending order.
std::vector<hicr_slot> distinct_slots(hicr_ctx c, const hicr_desc *d, uint64_t n) {
  std::vector<hicr_slot> sl;
  if (c->slots.size() <= 16 * n) {  // few slots: mark them (no sort of 2 n ids)
    std::vector<char> used(c->slots.size(), 0);
    for (uint64_t i = 0; i < n; i++) used[d[i].dst_slot] = used[d[i].src_slot] = 1;
    for (hicr_slot x = 0; x < used.size(); x++)
      if (used[x]) sl.push_back(x);
    return sl;
  }
  sl.reserve(2 * n);
  for (uint64_t i = 0; i < n; i++) {
    sl.push_back(d[i].dst_slot);
    sl.push_back(d[i].src_slot);
  }
  std::sort(sl.begin(), sl.end());
  sl.erase(std::unique(sl.begin(), sl.end()), sl.end());
  return sl;
}

// Share a stream plan out anew for the copy grid that is set now.
hipError_t recut(hicr_ctx c, hicr_plan p) {
  const int per_cu = c->grid_per_cu;
  if (!p->cuts.count(per_cu)) {
    const uint32_t w = p->share(per_cu);
    const StreamStart *at = nullptr;
    for (auto &k : p->cuts)
      if (k.second.first == w) at = k.second.second;
    if (!at) {
      std::vector<StreamStart> s(w + 1);
      stream_starts(p->h.data(), p->h.data() + p->n, p->n, p->bytes, w, kLineBytes, s.data(),
                    p->n_short);
      void *d = nullptr;
      p->more.reserve(p->more.size() + 1);
      hipError_t e = hipMalloc(&d, s.size() * sizeof s[0]);
      if (e != hipSuccess) return e;
      p->more.push_back(d);
      e = hipMemcpy(d, s.data(), s.size() * sizeof s[0], hipMemcpyHostToDevice);
      if (e != hipSuccess) return e;
      at = static_cast<const StreamStart *>(d);
    }
    p->cuts[per_cu] = {w, at};
  }
  std::tie(p->waves, p->starts) = p->cuts[per_cu];
  p->per_cu = per_cu;
  return hipSuccess;
}

int wait_plan(hicr_ctx c, hicr_plan p) {
  if (!p->launched) return HICR_OK;
  hipError_t e = wait_signal(c, p->sig);
  p->launched = false;
  return e == hipSuccess ? HICR_OK : hip_fail(c, e, "waiting for a plan replay");
}

}  // namespace

namespace hicr {

int wait_plans(hicr_ctx c) {
  int rc = HICR_OK;
  for (hicr_plan p : c->plans) {
    int r = wait_plan(c, p);
    if (r != HICR_OK) rc = r;
  }
  return rc;
}

bool plans_inflight(hicr_ctx c) {
  for (hicr_plan p : c->plans) {
    if (!p->launched) continue;
    if (!ended(c, p->sig)) return true;
    p->launched = false;
  }
  return false;
}

void plans_unfinished(hicr_ctx c, uint32_t slot, uint64_t *sent, uint64_t *recv) {
  for (hicr_plan p : c->plans) {
    if (!p->host_count || !p->launched || ended(c, p->sig)) continue;
    const uint64_t done = p->replays.ended(p->sig.words);
    const size_t k = std::lower_bound(p->slots.begin(), p->slots.end(), slot) - p->slots.begin();
    if (k == p->slots.size() || p->slots[k] != slot) continue;
    *sent -= (p->sig.seq - done) * p->n_sent[k];
    *recv -= (p->sig.seq - done) * p->n_recv[k];
  }
}

void destroy_plans(hicr_ctx c) {
  for (hicr_plan p : c->plans) {
    (void)wait_plan(c, p);
    free_plan(p);
  }
  c->plans.clear();
  for (void *b : c->plan_blocks) (void)hipHostFree(b);
  c->plan_blocks.clear();
  c->plan_words.clear();
}

}  // namespace hicr

extern "C" {

int hicr_plan_create(hicr_ctx c, const hicr_desc *d, uint64_t n, const hicr_sched *s,
                     uint32_t flags, hicr_plan *out, uint64_t *bad) {
  return guarded([&]() -> int {
    if (!c || !out || (n && !d) || (flags & ~HICR_PLAN_GRAPH)) return HICR_EINVAL;
    *out = nullptr;
    std::lock_guard<std::mutex> g(c->mu);
    (void)hipSetDevice(c->device);
    for (uint64_t i = 0; i < n; i++) {
      int rc = check_desc(c, d[i]);
      if (rc != HICR_OK) {
        if (bad) *bad = i;
        return fail(c, rc, "plan request %llu rejected", (unsigned long long)i);
      }
    }
    hicr_sched sched = s ? *s : c->def_sched;
    if (sched.mode == HICR_SCHED_TUNED || sched.mode == HICR_SCHED_LEARNED) {
      // resolved once, the network's class by the device forward kernel:
      // every replay uses the class chosen now
      int rc = choose_sched(c, d, n, sched.mode, &sched, true, flags & HICR_PLAN_GRAPH);
      if (rc != HICR_OK) return rc;
    } else if (sched.mode != HICR_SCHED_FIXED) {
      return fail(c, HICR_EINVAL, "unknown schedule mode %u", sched.mode);
    }
    int rc = check_sched(c, sched);
    if (rc != HICR_OK) return rc;

    hicr_plan p = new (std::nothrow) hicr_plan_s();
    if (!p) return HICR_ENOMEM;
    p->c = c;
    p->n = n;
    p->slots = distinct_slots(c, d, n);
    for (hicr_slot x : p->slots) c->slots[x].plan_refs++;

    constexpr size_t kHeadWords = hicr_plan_s::kHead / 8;
    std::vector<uint64_t> up(kHeadWords + 4 * n, 0);  // what goes to the device
    uint64_t *h = up.data() + kHeadWords;
    pack_batch(c, d, n, h);
    DevSched ds{sched.chunk_bytes, sched.wgs_per_desc, sched.unroll, 0};
    p->ds = ds;
    rc = split_batch(c, h, h + 2 * n, n, ds, p->segs);
    if (rc != HICR_OK) {
      free_plan(p);
      return rc;
    }
    // (a captured launch cannot number its replays: graphs count on the device)
    p->host_count = n && !(flags & HICR_PLAN_GRAPH) && writes_device_only(c, d, n);
    hipStream_t cs = nullptr;
    hipError_t e = hipEventCreateWithFlags(&p->sig.ev, hipEventDisableTiming);
    if (p->host_count) {
      p->n_sent.assign(p->slots.size(), 0);
      p->n_recv.assign(p->slots.size(), 0);
      for (uint64_t i = 0; i < n; i++) {
        c->slots[d[i].src_slot].tmp_sent++;
        c->slots[d[i].dst_slot].tmp_recv++;
        p->bytes += d[i].size;
        if (c->slots[d[i].src_slot].space != HICR_MEM_HBM) p->host_bytes += d[i].size;
        p->n_short += d[i].size < kStreamShort;
      }
      for (size_t k = 0; k < p->slots.size(); k++) {
        Slot &x = c->slots[p->slots[k]];
        p->n_sent[k] = x.tmp_sent;
        p->n_recv[k] = x.tmp_recv;
        x.tmp_sent = x.tmp_recv = 0;
      }
      p->per_cu = c->grid_per_cu;
      if (p->bytes <= stream_most(n, ds.chunk))
        p->waves = p->share(p->per_cu);
      if (p->waves) {
        static_assert(sizeof(StreamStart) == 16, "two words");
        up.resize(up.size() + 2 * (p->waves + 1));
        h = up.data() + kHeadWords;
        stream_starts(h, h + 2 * n, n, p->bytes, p->waves, kLineBytes,
                      reinterpret_cast<StreamStart *>(h + 4 * n), p->n_short);
        p->h.assign(h, h + n);
        p->h.insert(p->h.end(), h + 2 * n, h + 3 * n);
      }
      if (e == hipSuccess) e = take_words(c, &p->sig.words);
    }
    if (e == hipSuccess && n)
      e = hipMalloc(&p->d, std::max(hicr_plan_s::kHead + batch_bytes(n), up.size() * 8));
    if (e == hipSuccess && n) e = hipMemcpy(p->d, up.data(), up.size() * 8, hipMemcpyHostToDevice);
    p->sig.arrive = static_cast<uint32_t *>(p->d);
    if (p->waves && p->d) {
      p->starts = reinterpret_cast<const StreamStart *>(p->batch() + 4 * n);
      p->cuts[p->per_cu] = {p->waves, p->starts};
    }
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&cs, hipStreamNonBlocking);
    if (e != hipSuccess) {
      if (cs) (void)hipStreamDestroy(cs);
      free_plan(p);
      return hip_fail(c, e, "allocating a plan");
    }
    const uint64_t *dd = p->batch();
    uint32_t *tables = n ? batch_tables(p->batch(), n) : nullptr;
    // the piece tables are scanned once; every replay reads them
    if (!p->waves) rc = launch_scans(c, nullptr, dd, n, p->segs, ds, tables, cs);
    if (rc == HICR_OK) {
      e = hipStreamSynchronize(cs);
      if (e != hipSuccess) rc = hip_fail(c, e, "scanning a plan");
    }
    if (rc != HICR_OK) {
      (void)hipStreamDestroy(cs);
      free_plan(p);
      return rc;
    }
    if (flags & HICR_PLAN_GRAPH) {
      e = hipStreamBeginCapture(cs, hipStreamCaptureModeRelaxed);
      if (e == hipSuccess) {
        rc = launch_copies(c, dd, n, p->segs, ds, tables, c->d_counters, cs);
        hipGraph_t graph = nullptr;
        hipError_t e2 = hipStreamEndCapture(cs, &graph);
        p->graph = graph;
        if (rc == HICR_OK && e2 != hipSuccess) rc = hip_fail(c, e2, "capturing a plan");
        if (rc == HICR_OK) {
          e = hipGraphInstantiate(&p->exec, p->graph, nullptr, nullptr, 0);
          if (e != hipSuccess) rc = hip_fail(c, e, "instantiating a plan");
        }
      } else {
        rc = hip_fail(c, e, "capturing a plan");
      }
    }
    (void)hipStreamDestroy(cs);
    if (rc != HICR_OK) {
      free_plan(p);
      return rc;
    }
    c->plans.push_back(p);
    *out = p;
    return HICR_OK;
  });
}

int hicr_plan_launch(hicr_plan p, void *stream) {
  return guarded([&]() -> int {
    if (!p) return HICR_EINVAL;
    hicr_ctx c = p->c;
    std::lock_guard<std::mutex> g(c->mu);
    (void)hipSetDevice(c->device);
    hipStream_t s = stream ? static_cast<hipStream_t>(stream) : c->stream;
    hipError_t e = hipSuccess;
    if (p->launched && s != p->last) {
      e = ensure_event(c, p->sig);
      if (e == hipSuccess) e = hipStreamWaitEvent(s, p->sig.ev, 0);
    }
    if (e != hipSuccess) return hip_fail(c, e, "launching a plan");
    const uint64_t *dd = p->batch();
    // A captured launch is part of a graph of the caller's: it is counted on the
    // device, as often as that runs, and is no replay that a fence waits for.
    const bool cap = p->host_count && capturing(c, s), host_count = p->host_count && !cap;
    uint64_t *counters = host_count ? nullptr : c->d_counters;
    if (p->n && !host_count) c->dev_counted = true;
    // (without room for another cut the one there is serves as well)
    if (p->waves && p->per_cu != c->grid_per_cu && !cap && recut(c, p) != hipSuccess)
      (void)hipGetLastError();
    const uint64_t seq = p->sig.seq;
    const uint32_t n_words = p->sig.n_words;
    int rc = HICR_OK;
    if (p->exec) {
      e = hipGraphLaunch(p->exec, s);
    } else if (p->waves) {
      const DevBatch b{dd, dd + p->n, dd + 2 * p->n, dd + 3 * p->n, (uint32_t)p->n};
      e = launch_stream(b, p->starts, p->waves,
                        cap ? Done{} : arm(p->sig, stream_grid(p->waves)), s);
      if (e == hipSuccess && cap) rc = launch_counts(c, dd, p->n, counters, s, nullptr);
    } else if (p->n) {
      // replays are ordered (same stream, or the wait above), so the words'
      // last value is the last replay's
      rc = launch_copies(c, dd, p->n, p->segs, p->ds, batch_tables(p->batch(), p->n), counters, s,
                         host_count ? &p->sig : nullptr);
    }
    if (e != hipSuccess) rc = hip_fail(c, e, "launching a plan");
    if (rc != HICR_OK || cap) {  // no replay: the words stay with the one before
      p->sig.seq = seq;
      p->sig.n_words = n_words;
      return rc;
    }
    if (host_count) p->replays.queued(p->sig.seq, p->sig.n_words, !p->launched);
    e = mark(c, p->sig, s);
    if (e != hipSuccess) return hip_fail(c, e, "launching a plan");
    for (size_t k = 0; k < p->n_sent.size(); k++) {
      c->slots[p->slots[k]].sent += p->n_sent[k];
      c->slots[p->slots[k]].recv += p->n_recv[k];
    }
    p->launched = true;
    p->last = s;
    return HICR_OK;
  });
}

int hicr_plan_destroy(hicr_plan p) {
  return guarded([&]() -> int {
    if (!p) return HICR_EINVAL;
    hicr_ctx c = p->c;
    std::lock_guard<std::mutex> g(c->mu);
    (void)hipSetDevice(c->device);
    int rc = wait_plan(c, p);
    c->plans.erase(std::remove(c->plans.begin(), c->plans.end(), p), c->plans.end());
    free_plan(p);
    return rc;
  });
}

}  // extern "C"
