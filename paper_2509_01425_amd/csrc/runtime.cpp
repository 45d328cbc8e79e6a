// runtime.cpp -- host side of the communication-manager data path: context,
// slot table, request validation, fused-batch submission and fences.
//
// Slots (HiCR Sec. 3.1.3) live in a host table; requests are validated on
// the host, resolved to absolute device addresses and packed as a structure
// of arrays into pinned staging.  A small batch is copied by one launch that
// reads them there; a larger one is moved to device memory by a kernel in
// front and copied by one fused launch.  The last launch raises words in
// pinned memory that the fence polls, and the requests are counted in the host
// table (many-request batches: by a counter kernel, in device memory).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <functional>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "hicr.h"
#include "chan.h"
#include "internal.h"
#include "noalloc.h"
#include "runtime.h"

using namespace hicr;

namespace {

constexpr uint32_t kChunks[3] = {4u << 10, 64u << 10, 1u << 20};
constexpr uint32_t kWgs[2] = {1, 4};
constexpr uint32_t kUnroll[2] = {2, 4};

}  // namespace

namespace hicr {

int fail(hicr_ctx c, int code, const char *fmt, ...) {
  if (c) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    c->err = buf;
  }
  return code;
}

int hip_fail(hicr_ctx c, hipError_t e, const char *what) {
  return fail(c, HICR_EDEVICE, "%s: %s", what, hipGetErrorString(e));
}

int check_sched(hicr_ctx c, const hicr_sched &s) {
  if (s.chunk_bytes < kLineBytes || s.chunk_bytes > (1u << 30) || s.chunk_bytes % kLineBytes)
    return fail(c, HICR_EINVAL, "chunk_bytes %u: must be a multiple of 128 in [128, 1 GiB]",
                s.chunk_bytes);
  if (s.wgs_per_desc < 1 || s.wgs_per_desc > 64)
    return fail(c, HICR_EINVAL, "wgs_per_desc %u outside [1, 64]", s.wgs_per_desc);
  if (s.unroll != 2 && s.unroll != 4) return fail(c, HICR_EINVAL, "unroll %u not 2 or 4", s.unroll);
  return HICR_OK;
}

int check_desc(hicr_ctx c, const hicr_desc &d) {
  if (d.dst_slot >= c->slots.size() || !c->slots[d.dst_slot].live) return HICR_EBADSLOT;
  if (d.src_slot >= c->slots.size() || !c->slots[d.src_slot].live) return HICR_EBADSLOT;
  const Slot &ds = c->slots[d.dst_slot], &ss = c->slots[d.src_slot];
  if (d.dst_off > ds.size || d.size > ds.size - d.dst_off) return HICR_ERANGE;
  if (d.src_off > ss.size || d.size > ss.size - d.src_off) return HICR_ERANGE;
  if (!(c->pair_mask & HICR_PAIR(ds.space, ss.space))) return HICR_EUNSUPPORTED;
  return HICR_OK;
}

// A submission has ended: so has what was queued on its stream before it.
static void sub_ended(hicr_ctx c, Sub &s) {
  s.inflight = false;
  c->push_done = std::max(c->push_done, s.push_seq);
}

bool any_inflight(hicr_ctx c) {
  if (c->na_inflight) {
    if (hipEventQuery(c->na_ev) == hipSuccess)
      c->na_inflight = false;
    else
      return true;
  }
  bool any = false;
  for (Sub &s : c->subs) {
    if (s.inflight && ended(c, s.sig)) sub_ended(c, s);
    any = any || s.inflight;
  }
  return any;
}

hipError_t sync_event(hipEvent_t e) {
  // A fence usually waits for a few microseconds of GPU work: poll first
  // (hipEventSynchronize may sleep and wake tens of microseconds late), then
  // block, so a long wait does not burn a core.
  const auto t0 = std::chrono::steady_clock::now();
  for (;;) {
    const hipError_t q = hipEventQuery(e);
    if (q != hipErrorNotReady) return q;
    if (std::chrono::steady_clock::now() - t0 > std::chrono::microseconds(200)) break;
  }
  return hipEventSynchronize(e);
}

hipError_t mark(hicr_ctx c, Signal &sig, hipStream_t s) {
  sig.recorded = !(c->own_stream && s == c->stream);
  return sig.recorded ? hipEventRecord(sig.ev, s) : hipSuccess;
}

hipError_t ensure_event(hicr_ctx c, Signal &sig) {
  if (sig.recorded) return hipSuccess;
  const hipError_t e = hipEventRecord(sig.ev, c->stream);
  if (e == hipSuccess) sig.recorded = true;
  return e;
}

static bool raised(const Signal &sig) {
  for (uint32_t i = 0; i < sig.n_words; i++)
    if (__atomic_load_n(&sig.words[i], __ATOMIC_ACQUIRE) != sig.seq) return false;
  return sig.n_words != 0;
}

bool ended(hicr_ctx c, Signal &sig) {
  if (raised(sig)) return true;
  if (sig.n_words && !sig.recorded) return false;
  return ensure_event(c, sig) == hipSuccess && hipEventQuery(sig.ev) == hipSuccess;
}

hipError_t wait_signal(hicr_ctx c, Signal &sig) {
  if (sig.n_words) {
    const auto t0 = std::chrono::steady_clock::now();
    for (uint32_t k = 0;; k++) {
      if (raised(sig)) return hipSuccess;
      if ((k & 15) == 15 && std::chrono::steady_clock::now() - t0 > std::chrono::microseconds(200))
        break;
    }
  }
  const hipError_t e = ensure_event(c, sig);
  return e == hipSuccess ? sync_event(sig.ev) : e;
}

bool capturing(hicr_ctx c, hipStream_t s) {
  if (c->own_stream && s == c->stream) return false;
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &st) == hipSuccess) return st == hipStreamCaptureStatusActive;
  (void)hipGetLastError();
  return false;
}

bool writes_device_only(hicr_ctx c, const hicr_desc *d, uint64_t n) {
  for (uint64_t i = 0; i < n; i++)
    if (c->slots[d[i].dst_slot].space != HICR_MEM_HBM) return false;
  return true;
}

bool same_under_every_class(hicr_ctx c, const hicr_desc *d, uint64_t n) {
  if (n > kStreamMaxReqs) return false;
  const uint64_t most = stream_most(n, 0);
  uint64_t bytes = 0;
  for (uint64_t i = 0; i < n; i++) {
    if (d[i].dst_slot >= c->slots.size() || c->slots[d[i].dst_slot].space != HICR_MEM_HBM ||
        d[i].size > most)
      return false;
    bytes += d[i].size;
  }
  return bytes <= most;
}

int wait_sub(hicr_ctx c, Sub &s) {
  if (!s.inflight) return HICR_OK;
  hipError_t e = wait_signal(c, s.sig);
  sub_ended(c, s);
  if (e != hipSuccess) return hip_fail(c, e, "waiting for a batch");
  return HICR_OK;
}

int wait_all(hicr_ctx c) {
  int rc = HICR_OK;
  for (Sub &s : c->subs) {
    int r = wait_sub(c, s);
    if (r != HICR_OK) rc = r;
  }
  if (c->na_inflight) {
    hipError_t e = sync_event(c->na_ev);
    c->na_inflight = false;
    c->na_up_pending = false;  // the upload precedes the launches on one stream
    if (e != hipSuccess) rc = hip_fail(c, e, "waiting for a no-allocation batch");
  }
  int r = wait_extra(c);
  if (r != HICR_OK) rc = r;
  r = wait_plans(c);
  if (r != HICR_OK) rc = r;
  return rc;
}

// Room for n requests in a submission buffer's staging, and on the device
// (for the piece kernels).
static uint64_t grown(uint64_t cap, uint64_t n) {
  return std::max<uint64_t>(n, std::max<uint64_t>(2 * cap, 4096));
}
static int ensure_staging(hicr_ctx c, Sub &s, uint64_t n) {
  if (n <= s.h_cap) return HICR_OK;
  const uint64_t cap = grown(s.h_cap, n);
  if (s.h && s.h_cap > kStageReqs) (void)hipHostFree(s.h);
  s.h = nullptr;
  s.h_cap = 0;
  hipError_t e = hipHostMalloc(&s.h, stage_bytes(cap), hipHostMallocDefault);
  if (e == hipSuccess) e = hipHostGetDevicePointer(&s.h_dev, s.h, 0);
  if (e != hipSuccess) return fail(c, HICR_ENOMEM, "pinned staging of %llu requests", (unsigned long long)cap);
  s.h_cap = cap;
  return HICR_OK;
}
static int ensure_device(hicr_ctx c, Sub &s, uint64_t n) {
  if (n <= s.d_cap) return HICR_OK;
  const uint64_t cap = grown(s.d_cap, n);
  if (s.d) (void)hipFree(s.d);
  s.d = nullptr;
  s.d_cap = 0;
  if (hipMalloc(&s.d, batch_bytes(cap)) != hipSuccess) {
    s.d = nullptr;
    return fail(c, HICR_ENOMEM, "device batch buffer of %llu requests", (unsigned long long)cap);
  }
  s.d_cap = cap;
  return HICR_OK;
}

// The counter table is allocated once, for kMaxSlots slots (16 MiB), so its
// address never changes: captured plans keep a valid pointer to it.  The
// submission buffers' and the pushes' arrival counters lie behind it.
static int alloc_counters(hicr_ctx c) {
  const size_t bytes = (size_t)kMaxSlots * 16 + 128 * (kNumSubs + 1);
  hipError_t e = hipMalloc(&c->d_counters, bytes);
  if (e == hipSuccess) e = hipMemset(c->d_counters, 0, bytes);
  if (e != hipSuccess) return hip_fail(c, e, "allocating the counter table");
  c->counter_cap = kMaxSlots;
  uint32_t *arrive = reinterpret_cast<uint32_t *>(c->d_counters + 2 * (size_t)kMaxSlots);
  for (int i = 0; i < kNumSubs; i++) c->subs[i].sig.arrive = arrive + 32 * i;
  c->push_sig.arrive = arrive + 32 * kNumSubs;
  return HICR_OK;
}

// Copy workgroups per CU when the caller has not fixed it.  Measured on the
// batched workload (256 CUs): with 64 KiB or 1 MiB pieces two workgroups per
// CU (eight wavefronts, each with two rounds of `unroll` 1 KiB rows in
// flight) are the fastest at either unroll, 1-2 % above one or four; 4 KiB
// pieces spend more time per piece on the search and want four.  32 KiB
// pieces at unroll 4 run 1.7 % faster with one workgroup per CU than with
// two (0.6-1 % on 64 MiB copies, aligned or not); 24 KiB pieces tie, 48 KiB
// pieces lose 0.6 %.  Pieces of 16 KiB or less get at least four from the
// latency rule in launch_copies.
int default_grid_per_cu(const DevSched &ds) {
  if (ds.chunk <= (4u << 10)) return 4;
  if (ds.chunk <= (32u << 10)) return 1;
  return 2;
}

int split_batch(hicr_ctx c, const uint64_t *hd, const uint64_t *hz, uint64_t n, const DevSched &ds,
                std::vector<Seg> &out) {
  out.clear();
  const bool lds = n <= kMaxLdsDescs;
  if (!lds) {
    // A piece spans at least 128 destination bytes except at a request's
    // ends, so a request has at most size / 128 + 2 pieces.  When that bound
    // keeps the batch under 2^31 pieces, no per-request count is needed on
    // the host (the scan kernel counts): launches split by request count
    // only, and `pieces` holds the lower bound, one per request.
    uint64_t bytes = 0;
    for (uint64_t i = 0; i < n; i++) bytes += hz[i];
    if (bytes < (1ull << 38) && (bytes >> 7) + 2 * n < (1ull << 31)) {
      const uint64_t cap = (uint64_t)kTile * kMaxTiles;
      for (uint64_t i0 = 0; i0 < n; i0 += cap) {
        const uint64_t i1 = std::min(n, i0 + cap);
        uint64_t b = bytes;
        if (i0 > 0 || i1 < n) {
          b = 0;
          for (uint64_t i = i0; i < i1; i++) b += hz[i];
        }
        out.push_back(Seg{i0, i1, i1 - i0, b, false});
      }
      return HICR_OK;
    }
  }
  uint64_t i0 = 0;
  while (i0 < n) {
    uint64_t i1 = i0, pieces = 0, bytes = 0;
    const uint64_t cap = lds ? kMaxLdsDescs : (uint64_t)kTile * kMaxTiles;
    while (i1 < n && i1 - i0 < cap) {
      uint64_t p = piece_count(hd[i1], hz[i1], ds.chunk, ds.wgs);
      if (i1 > i0 && pieces + p >= (1ull << 31)) break;
      pieces += p;
      bytes += hz[i1];
      i1++;
    }
    if (pieces >= (1ull << 31))
      return fail(c, HICR_EINVAL, "request %llu needs more than 2^31 pieces",
                  (unsigned long long)i0);
    out.push_back(Seg{i0, i1, pieces, bytes, lds});
    i0 = i1;
  }
  return HICR_OK;
}

static DevBatch seg_batch(const uint64_t *dd, uint64_t n, const Seg &g) {
  return DevBatch{dd + g.i0, dd + n + g.i0, dd + 2 * n + g.i0, dd + 3 * n + g.i0,
                  (uint32_t)(g.i1 - g.i0)};
}

int launch_scans(hicr_ctx c, const uint64_t *staged, const uint64_t *dd, uint64_t n,
                 const std::vector<Seg> &segs, DevSched ds, uint32_t *tables, hipStream_t stream) {
  for (const Seg &g : segs) {
    if (g.lds) continue;
    DevBatch from;
    if (staged) from = seg_batch(staged, n, g);
    hipError_t e = launch_scan(staged ? &from : nullptr, seg_batch(dd, n, g), ds, tables + g.i0,
                               tables + n + g.i0, stream);
    if (e != hipSuccess) return hip_fail(c, e, "launching the scan kernel");
  }
  return HICR_OK;
}

int launch_counts(hicr_ctx c, const uint64_t *dd, uint64_t n, uint64_t *counters,
                         hipStream_t stream, Signal *sig) {
  if (!counters || !n) return HICR_OK;
  Done done;
  if (sig) done = arm(*sig, count_grid(n));
  hipError_t e = launch_count(dd + 3 * n, n, counters, done, stream);
  return e == hipSuccess ? HICR_OK : hip_fail(c, e, "launching the counter kernel");
}

constexpr uint64_t kTableReqs = 12;  // of a scanned table, to a wave

int launch_copies(hicr_ctx c, const uint64_t *dd, uint64_t n, const std::vector<Seg> &segs,
                  DevSched ds, const uint32_t *tables, uint64_t *counters, hipStream_t stream,
                  Signal *sig) {
  const int per_cu_class = c->grid_per_cu > 0 ? c->grid_per_cu : default_grid_per_cu(ds);
  for (const Seg &g : segs) {
    // A launch over a scanned table whose pieces average under 16 KiB (a
    // halo exchange's rows) takes four groups per CU: 151.6 us an exchange
    // against 153.4 with two, 149.6 with eight.  (With an LDS table every
    // group re-scans the batch, so more groups cost more there.)
    int per_cu = per_cu_class;
    if (c->grid_per_cu == 0 && !g.lds &&
        (ds.chunk <= (16u << 10) || g.bytes < (g.i1 - g.i0) * (16u << 10)))
      per_cu = std::max(per_cu, 4);
    if (g.lds) per_cu = std::min(per_cu, c->occ);
    uint64_t cap_grid = (uint64_t)c->n_cu * (uint64_t)per_cu;
    // ... of at least 16 KiB or kTableReqs requests a wavefront (7,744 rows of
    // 2,816 B: 19 us a replay that way, 24 us with four groups per CU; 5,000 of
    // 16 B 415 us by bytes alone, now 15; 20,000 of 1 KiB 25 us with 6 requests,
    // 24 with 8, 22 with 12)
    if (c->grid_per_cu == 0 && !g.lds)
      cap_grid = std::min(cap_grid, std::max(g.bytes >> 16, (g.i1 - g.i0) / (4 * kTableReqs) + 1));
    // every wavefront of a workgroup copies its own pieces
    const uint64_t want = (g.pieces + kCopyBlock / 64 - 1) / (kCopyBlock / 64);
    const uint32_t grid = (uint32_t)std::min<uint64_t>(std::max<uint64_t>(want, 1), cap_grid);
    // the last launch of the submission tells of its end (the launches of one
    // stream run one after another)
    const bool tell = sig && !counters && &g == &segs.back();
    hipError_t e;
    if (g.lds) {
      e = launch_copy(seg_batch(dd, n, g), ds, grid, stream);
      if (e == hipSuccess && tell) e = launch_done(arm(*sig, 1), stream);
    } else {
      Done done;
      if (tell) done = arm(*sig, grid);
      e = launch_copy_mem(seg_batch(dd, n, g), ds, tables + g.i0, tables + n + g.i0, grid, done,
                          stream);
    }
    if (e != hipSuccess) return hip_fail(c, e, "launching the copy kernel");
  }
  return launch_counts(c, dd, n, counters, stream, sig);
}

// Host threads for batches large enough that validating and packing them on
// one core would take longer than their copy (a halo exchange: 61,952
// requests, 130 us on one core).  run(blocks, f) calls f(block) for every block
// in [0, blocks) and returns when all are done.  The calling thread takes
// blocks from the start; a pool thread joins in once it is awake (50-100 us
// after it is called) and is not waited for if nothing is left by then:
// the halo exchange 326 us a pass with three threads waited for, 307 with three
// that join in, 257 with seven, 336 without any.
class HostPool {
 public:
  explicit HostPool(int extra) {
    try {
      for (int i = 0; i < extra; i++) th_.emplace_back([this] { loop(); });
    } catch (...) {
      stop();  // join the threads already started, then report the failure
      throw;
    }
  }
  ~HostPool() { stop(); }
  int size() const { return (int)th_.size() + 1; }
  void run(uint32_t blocks, const std::function<void(uint32_t)> &f) {
    {
      std::lock_guard<std::mutex> g(m_);
      f_ = &f;
      blocks_ = blocks;
      next_ = 0;
      gen_++;
    }
    cv_.notify_all();
    work(f, blocks);
    std::unique_lock<std::mutex> g(m_);
    f_ = nullptr;  // who wakes up from here on finds nothing to do
    done_.wait(g, [&] { return active_ == 0; });
  }

 private:
  void stop() {
    {
      std::lock_guard<std::mutex> g(m_);
      quit_ = true;
    }
    cv_.notify_all();
    for (std::thread &t : th_)
      if (t.joinable()) t.join();
  }
  void work(const std::function<void(uint32_t)> &f, uint32_t blocks) {
    for (uint32_t b; (b = next_.fetch_add(1, std::memory_order_relaxed)) < blocks;) f(b);
  }
  void loop() {
    uint64_t seen = 0;
    std::unique_lock<std::mutex> g(m_);
    for (;;) {
      cv_.wait(g, [&] { return quit_ || gen_ != seen; });
      if (quit_) return;
      seen = gen_;
      if (!f_) continue;
      const std::function<void(uint32_t)> &f = *f_;
      const uint32_t blocks = blocks_;
      active_++;
      g.unlock();
      work(f, blocks);
      g.lock();
      if (--active_ == 0) done_.notify_one();
    }
  }
  std::vector<std::thread> th_;
  std::mutex m_;
  std::condition_variable cv_, done_;
  const std::function<void(uint32_t)> *f_ = nullptr;
  std::atomic<uint32_t> next_{0};
  uint32_t blocks_ = 0;
  uint64_t gen_ = 0;
  int active_ = 0;
  bool quit_ = false;
};

void destroy_pool(hicr_ctx c) {
  delete c->pool;
  c->pool = nullptr;
}

constexpr uint64_t kPoolMin = 16384;        // requests that make a batch large
constexpr uint64_t kPackBlock = 2048;       // requests a host thread takes at once
constexpr int kPoolThreads = 7;             // beside the calling one
constexpr uint64_t kUploadStream = 256 << 10;  // upload bytes that go on their own stream

// What pack_range found: the first rejected request (i1 if none) and its
// code, the bytes of all and of those read from host memory, how many are short
// (stream_load), and whether one writes host memory.
struct Packed {
  uint64_t bad = 0;
  int rc = HICR_OK;
  uint64_t bytes = 0, host_bytes = 0, n_short = 0;
  bool host_dst = false;
};

// Validate requests [i0, i1) of n and resolve them to the structure of arrays
// {dst, src, size, slot pair}.
static Packed pack_range(hicr_ctx c, const hicr_desc *d, uint64_t n, uint64_t i0, uint64_t i1,
                         uint64_t *h) {
  uint64_t *hd = h, *hs = h + n, *hz = h + 2 * n, *hp = h + 3 * n;
  const Slot *sl = c->slots.data();
  Packed p;
  p.bad = i1;
  // (not in p: they would be stored for every request)
  uint64_t bytes = 0, host_bytes = 0, n_short = 0;
  uint32_t to = 0;  // spaces
  for (uint64_t i = i0; i < i1; i++) {
    const hicr_desc &x = d[i];
    const int rc = check_desc(c, x);
    if (rc != HICR_OK) {
      p.rc = rc;
      p.bad = i;
      return p;
    }
    hd[i] = sl[x.dst_slot].base + x.dst_off;
    hs[i] = sl[x.src_slot].base + x.src_off;
    hz[i] = x.size;
    hp[i] = (uint64_t)x.dst_slot | ((uint64_t)x.src_slot << 32);
    bytes += x.size;
    n_short += x.size < kStreamShort;
    to |= sl[x.dst_slot].space;
    host_bytes += x.size & (0 - (uint64_t)(sl[x.src_slot].space != HICR_MEM_HBM));
  }
  static_assert(HICR_MEM_HBM == 0, "any other space of a destination shows");
  p.bytes = bytes;
  p.host_bytes = host_bytes;
  p.n_short = n_short;
  p.host_dst = to != HICR_MEM_HBM;
  return p;
}

void pack_batch(hicr_ctx c, const hicr_desc *d, uint64_t n, uint64_t *h) {
  (void)pack_range(c, d, n, 0, n, h);
}

// The same for the whole batch, split over host threads when it is large.
static Packed pack_all(hicr_ctx c, const hicr_desc *d, uint64_t n, uint64_t *h) {
  if (n < kPoolMin || !c->pool || c->pool->size() == 1) return pack_range(c, d, n, 0, n, h);
  const uint32_t blocks = (uint32_t)((n + kPackBlock - 1) / kPackBlock);
  std::vector<Packed> part(blocks);
  c->pool->run(blocks, [&](uint32_t p) {
    part[p] = pack_range(c, d, n, p * kPackBlock, std::min(n, (p + 1) * kPackBlock), h);
  });
  Packed k;
  k.bad = n;
  for (uint32_t p = blocks; p-- > 0;) {
    k.bytes += part[p].bytes;
    k.host_dst |= part[p].host_dst;
    if (part[p].rc != HICR_OK) {
      k.bad = part[p].bad;
      k.rc = part[p].rc;
    }
  }
  return k;
}

// Start the pool behind a context's first large batch, while that one is on
// the GPU (starting seven threads takes longer than packing it alone).
static void start_pool(hicr_ctx c, uint64_t n) {
  if (n < kPoolMin || c->pool || c->pool_failed) return;
  // no exception crosses the C ABI: a pool that cannot start its threads
  // leaves the work on the calling thread
  try {
    const int hw = (int)std::thread::hardware_concurrency();
    c->pool = new HostPool(std::max(0, std::min(kPoolThreads, hw - 1)));
  } catch (...) {
    c->pool = nullptr;
    c->pool_failed = true;
  }
}

// Validate, pack and launch n requests as one submission.
int submit(hicr_ctx c, const hicr_desc *d, uint64_t n, const hicr_sched &sched,
           hipStream_t stream, uint64_t *bad, const SubmitOpts *opt) {
  if (n == 0) return HICR_OK;
  // Choose the submission buffer (round robin; wait if still in flight).
  Sub &s = c->subs[c->next_sub];
  c->next_sub = (c->next_sub + 1) % kNumSubs;
  int rc = wait_sub(c, s);
  if (rc != HICR_OK) return rc;
  rc = ensure_staging(c, s, n);
  if (rc != HICR_OK) return rc;
  uint64_t *h = static_cast<uint64_t *>(s.h);
  const uint64_t *hv = static_cast<const uint64_t *>(s.h_dev);  // the same, as the device sees it
  // nothing is queued unless every request passes
  const Packed k = pack_all(c, d, n, h);
  if (k.rc != HICR_OK) {
    if (bad) *bad = k.bad;
    return fail(c, k.rc, "request %llu rejected", (unsigned long long)k.bad);
  }
  // How the end is seen and the requests are counted.  A batch into HBM of at
  // most kMaxLdsDescs requests is counted here, in its slots, and its last
  // copy launch raises the submission's words; a larger one is counted on the
  // device by a kernel that raises them (a host core takes ~2 ns a request);
  // bytes in host memory are only visible after the runtime's completion
  // signal, so there the event tells.  Work that a caller captures runs as
  // often as its graph is launched: it is counted on the device.
  const bool no_count = opt && opt->no_count, cap = capturing(c, stream);
  const bool host_count = !no_count && !k.host_dst && !cap && n <= kMaxLdsDescs;
  uint64_t *counters = no_count || host_count ? nullptr : c->d_counters;
  Signal *sig = k.host_dst || opt || cap ? nullptr : &s.sig;
  const uint32_t waves =
      k.host_dst || opt || k.bytes > stream_most(n, sched.chunk_bytes)
          ? 0
          : stream_waves(n, k.bytes, c->n_cu, c->grid_per_cu, k.n_short, 2 * k.host_bytes > k.bytes);
  s.sig.n_words = 0;
  s.host_counted = 0;
  hipError_t e = hipSuccess;
  if (waves) {
    const Done done = sig ? arm(*sig, stream_grid(waves)) : Done{};
    const uint64_t load = k.bytes + k.n_short * kStreamExtra;
    uint64_t dst, src;
    if (args_fit(h, n, load, &dst, &src)) {
      e = launch_stream_args(h, (uint32_t)n, dst, src, load, waves, done, stream);
    } else {
      // small enough that the kernel reads the requests where they are
      StreamStart *starts = reinterpret_cast<StreamStart *>(h + 4 * n);
      stream_starts(h, h + 2 * n, n, k.bytes, waves, kLineBytes, starts, k.n_short);
      const DevBatch b{hv, hv + n, hv + 2 * n, hv + 3 * n, (uint32_t)n};
      e = launch_stream(b, reinterpret_cast<const StreamStart *>(hv + 4 * n), waves, done, stream);
    }
    rc = e == hipSuccess ? launch_counts(c, hv, n, counters, stream, nullptr)
                         : hip_fail(c, e, "launching the stream kernel");
  } else {
    const DevSched ds{sched.chunk_bytes, sched.wgs_per_desc, sched.unroll, 0};
    rc = ensure_device(c, s, n);
    if (rc == HICR_OK) rc = split_batch(c, h, h + 2 * n, n, ds, c->segs);
    if (rc != HICR_OK) return rc;
    const uint64_t *dd = static_cast<const uint64_t *>(s.d);
    uint32_t *tables = batch_tables(s.d, n);
    const bool lds = c->segs[0].lds;  // all of them, or none
    // A large batch behind others still in flight is uploaded on a stream of
    // its own, so the upload overlaps their copies.  Otherwise a kernel in
    // front of the copy reads the staging (the scan kernel, when there is a
    // table to scan): a copy engine first waits for the signal of the kernel
    // before it, and the copy kernel then for the engine's.  A timed submission
    // is uploaded before the first event in any case.
    const bool behind = !cap && n * 32 >= kUploadStream && any_inflight(c);
    if (behind) {
      e = hipMemcpyAsync(s.d, s.h, n * 32, hipMemcpyHostToDevice, c->up);
      if (e == hipSuccess) e = hipEventRecord(s.up_ev, c->up);
      if (e == hipSuccess) e = hipStreamWaitEvent(stream, s.up_ev, 0);
    } else if (lds || opt) {
      e = launch_upload(s.h_dev, s.d, n * (counters ? 32 : 24), stream);
    }
    if (e != hipSuccess) return hip_fail(c, e, "uploading a batch");
    if (opt && opt->t0) {
      e = hipEventRecord(opt->t0, stream);
      if (e != hipSuccess) return hip_fail(c, e, "recording a timing event");
    }
    rc = launch_scans(c, behind || lds || opt ? nullptr : hv, dd, n, c->segs, ds, tables, stream);
    if (rc == HICR_OK) rc = launch_copies(c, dd, n, c->segs, ds, tables, counters, stream, sig);
    if (rc == HICR_OK && opt && opt->t1) {
      e = hipEventRecord(opt->t1, stream);
      if (e != hipSuccess) rc = hip_fail(c, e, "recording a timing event");
    }
  }
  if (counters) c->dev_counted = true;
  // the staging buffer is in use from the first launch on, whatever failed
  // after it (then only the event tells when it is free again)
  if (rc != HICR_OK) s.sig.n_words = 0;
  e = mark(c, s.sig, stream);
  s.push_seq = stream == c->stream ? c->push_seq : 0;
  if (e == hipSuccess) s.inflight = true;
  start_pool(c, n);
  if (rc != HICR_OK) return rc;
  if (host_count) {
    const uint64_t *hp = h + 3 * n;
    for (uint64_t i = 0; i < n; i++) {
      c->slots[hp[i] & 0xffffffffull].recv++;
      c->slots[hp[i] >> 32].sent++;
    }
    s.host_counted = n;
  }
  if (e != hipSuccess) return hip_fail(c, e, "recording a batch event");
  return HICR_OK;
}

int flush_pending(hicr_ctx c) {
  if (c->pending.empty()) return HICR_OK;
  std::vector<hicr_desc> p;
  p.swap(c->pending);
  uint64_t bad = 0;
  return submit(c, p.data(), p.size(), c->def_sched, c->stream, &bad, nullptr);
}

}  // namespace hicr

// ---------------------------------------------------------------- C ABI

extern "C" {

int hicr_sched_class(uint32_t cls, hicr_sched *out) {
  return guarded([&]() -> int {
    if (!out || cls >= HICR_NUM_CLASSES) return HICR_EINVAL;
    out->chunk_bytes = kChunks[cls / 4];
    out->wgs_per_desc = kWgs[(cls / 2) % 2];
    out->unroll = kUnroll[cls % 2];
    out->mode = HICR_SCHED_FIXED;
    return HICR_OK;
  });
}

const char *hicr_strerror(int code) {
  switch (code) {
    case HICR_OK: return "ok";
    case HICR_EINVAL: return "invalid argument";
    case HICR_ERANGE: return "offset or size outside the slot";
    case HICR_EBADSLOT: return "unknown or deregistered slot";
    case HICR_EUNSUPPORTED: return "memory-space pair not supported";
    case HICR_EAGAIN: return "channel full or empty; try again";
    case HICR_ENOMEM: return "out of memory";
    case HICR_ETIMEDOUT: return "timed out";
    case HICR_EHAZARD: return "conflicting requests in one epoch";
    case HICR_EDEVICE: return "device or HIP runtime error";
    case HICR_EBUSY: return "transfers still in flight";
    default: return "unknown error";
  }
}

int hicr_last_error(hicr_ctx c, char *buf, size_t n) {
  return guarded([&]() -> int {
    if (!c || !buf || n == 0) return HICR_EINVAL;
    std::lock_guard<std::mutex> g(c->mu);
    snprintf(buf, n, "%s", c->err.c_str());
    return HICR_OK;
  });
}

int hicr_ctx_create(int device, void *stream, hicr_ctx *out) {
  return guarded([&]() -> int {
    if (!out) return HICR_EINVAL;
    *out = nullptr;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) return HICR_EINVAL;
    if (hipSetDevice(device) != hipSuccess) return HICR_EDEVICE;
    hicr_ctx c = new (std::nothrow) hicr_ctx_s();
    if (!c) return HICR_ENOMEM;
    c->device = device;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) != hipSuccess) {
      delete c;
      return HICR_EDEVICE;
    }
    c->n_cu = prop.multiProcessorCount;
    if (copy_occupancy(&c->occ) != 0 || c->occ < 1) c->occ = 1;
    if (stream) {
      c->stream = static_cast<hipStream_t>(stream);
      c->own_stream = false;
    } else if (hipStreamCreateWithFlags(&c->stream, hipStreamNonBlocking) != hipSuccess) {
      delete c;
      return HICR_EDEVICE;
    } else {
      c->own_stream = true;
    }
    bool ok = hipStreamCreateWithFlags(&c->aux, hipStreamNonBlocking) == hipSuccess;
    ok = ok && hipHostMalloc(&c->h_read, 64, hipHostMallocDefault) == hipSuccess;
    // pinned, in one block: the submission buffers' done words, their staging
    // for kStageReqs requests each (larger submissions allocate their own),
    // and the staging of hicr_memcpy_batch_noalloc
    constexpr size_t done_bytes = 4096, na_bytes = kNoAllocMaxReqs * 32;
    static_assert(8 * kDoneWords * kNumSubs <= done_bytes, "one page of words");
    void *pinned = nullptr, *pinned_dev = nullptr;
    ok = ok && hipHostMalloc(&pinned, done_bytes + kNumSubs * stage_bytes(kStageReqs) + na_bytes,
                             hipHostMallocDefault) == hipSuccess;
    c->h_done = static_cast<uint64_t *>(pinned);
    ok = ok && hipHostGetDevicePointer(&pinned_dev, pinned, 0) == hipSuccess;
    if (ok) std::memset(c->h_done, 0, done_bytes);
    for (int i = 0; ok && i < kNumSubs; i++) {
      const size_t off = done_bytes + i * stage_bytes(kStageReqs);
      c->subs[i].h = static_cast<char *>(pinned) + off;
      c->subs[i].h_dev = static_cast<char *>(pinned_dev) + off;
      c->subs[i].h_cap = kStageReqs;
    }
    if (ok) c->na_h = static_cast<char *>(pinned) + done_bytes + kNumSubs * stage_bytes(kStageReqs);
    ok = ok && hipEventCreateWithFlags(&c->push_sig.ev, hipEventDisableTiming) == hipSuccess;
    if (ok && (pump_occupancy(&c->pump_occ) != 0 || c->pump_occ < 1)) c->pump_occ = 1;
    ok = ok && hipStreamCreateWithFlags(&c->up, hipStreamNonBlocking) == hipSuccess;
    for (int i = 0; ok && i < kNumSubs; i++) {
      c->subs[i].sig.words = c->h_done + kDoneWords * i;
      ok = hipEventCreateWithFlags(&c->subs[i].sig.ev, hipEventDisableTiming) == hipSuccess;
      ok = ok && hipEventCreateWithFlags(&c->subs[i].up_ev, hipEventDisableTiming) == hipSuccess;
    }
    c->def_sched = hicr_sched{64u << 10, 1, 2, HICR_SCHED_FIXED};
    // what hicr_memcpy_batch_noalloc needs, set up once here: the device
    // workspace's address, pinned staging, its events, and room for its
    // launch list and error messages (so that no call of it allocates)
    ok = ok && noalloc_scratch(device, &c->na_scratch) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&c->na_up_ev, hipEventDisableTiming) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&c->na_ev, hipEventDisableTiming) == hipSuccess;
    if (ok) {
      c->segs.reserve(kNoAllocSegCap);
      c->err.reserve(512);
    }
    if (!ok || alloc_counters(c) != HICR_OK) {
      hicr_ctx_destroy(c);
      return HICR_EDEVICE;
    }
    *out = c;
    return HICR_OK;
  });
}

int hicr_ctx_destroy(hicr_ctx c) {
  return guarded([&]() -> int {
    if (!c) return HICR_EINVAL;
    (void)hipSetDevice(c->device);
    wait_all(c);
    destroy_plans(c);
    destroy_extra(c);
    destroy_pump_bufs(c);
    destroy_sched(c);
    destroy_pool(c);
    for (Sub &s : c->subs) {
      if (s.h && s.h_cap > kStageReqs) (void)hipHostFree(s.h);
      if (s.d) (void)hipFree(s.d);
      if (s.sig.ev) (void)hipEventDestroy(s.sig.ev);
      if (s.up_ev) (void)hipEventDestroy(s.up_ev);
    }
    if (c->d_counters) (void)hipFree(c->d_counters);
    if (c->pp_d) (void)hipFree(c->pp_d);
    if (c->pp_h) (void)hipHostFree(c->pp_h);
    if (c->h_read) (void)hipHostFree(c->h_read);
    if (c->h_done) (void)hipHostFree(c->h_done);
    if (c->na_up_ev) (void)hipEventDestroy(c->na_up_ev);
    if (c->na_ev) (void)hipEventDestroy(c->na_ev);
    for (hipStream_t s : c->serve_streams) (void)hipStreamDestroy(s);
    if (c->aux) (void)hipStreamDestroy(c->aux);
    if (c->up) (void)hipStreamDestroy(c->up);
    if (c->own_stream && c->stream) (void)hipStreamDestroy(c->stream);
    delete c;
    return HICR_OK;
  });
}

int hicr_ctx_set_sched(hicr_ctx c, const hicr_sched *s) {
  return guarded([&]() -> int {
    if (!c || !s) return HICR_EINVAL;
    std::lock_guard<std::mutex> g(c->mu);
    if (s->mode != HICR_SCHED_FIXED) return fail(c, HICR_EINVAL, "default schedule must be fixed");
    int rc = check_sched(c, *s);
    if (rc == HICR_OK) c->def_sched = *s;
    return rc;
  });
}

int hicr_ctx_set_copy_grid(hicr_ctx c, uint32_t wgs_per_cu) {
  return guarded([&]() -> int {
    if (!c || wgs_per_cu > 64) return HICR_EINVAL;
    std::lock_guard<std::mutex> g(c->mu);
    c->grid_per_cu = (int)wgs_per_cu;
    return HICR_OK;
  });
}

int hicr_ctx_set_pairs(hicr_ctx c, uint32_t pair_mask) {
  return guarded([&]() -> int {
    if (!c || (pair_mask & ~HICR_PAIRS_ALL)) return HICR_EINVAL;
    std::lock_guard<std::mutex> g(c->mu);
    c->pair_mask = pair_mask;
    return HICR_OK;
  });
}

int hicr_slot_register(hicr_ctx c, void *ptr, uint64_t size, uint32_t memspace, hicr_slot *out) {
  return guarded([&]() -> int {
    if (!c || !out) return HICR_EINVAL;
    std::lock_guard<std::mutex> g(c->mu);
    (void)hipSetDevice(c->device);
    if (!ptr) return fail(c, HICR_EINVAL, "null address");
    if (size == 0) return fail(c, HICR_EINVAL, "a slot needs a non-zero size");
    if (memspace != HICR_MEM_HBM && memspace != HICR_MEM_HOST)
      return fail(c, HICR_EINVAL, "unknown memory space %u", memspace);
    if (memspace == HICR_MEM_HBM) {
      hipPointerAttribute_t attr;
      if (hipPointerGetAttributes(&attr, ptr) != hipSuccess || attr.type != hipMemoryTypeDevice ||
          attr.device != c->device) {
        (void)hipGetLastError();
        return fail(c, HICR_EINVAL, "address is not device memory of device %d", c->device);
      }
      hipDeviceptr_t base = nullptr;
      size_t alloc = 0;
      if (hipMemGetAddressRange(&base, &alloc, ptr) != hipSuccess) {
        (void)hipGetLastError();
        return fail(c, HICR_EINVAL, "address outside every device allocation");
      }
      uint64_t b = reinterpret_cast<uint64_t>(base), p = reinterpret_cast<uint64_t>(ptr);
      if (p - b > alloc || size > alloc - (p - b))
        return fail(c, HICR_ERANGE, "slot extends past the end of its allocation");
    }
    uint64_t dev_addr = reinterpret_cast<uint64_t>(ptr);
    if (memspace == HICR_MEM_HOST) {
      // pinned host memory: the device reaches it at its device-side address
      hipPointerAttribute_t attr;
      if (hipPointerGetAttributes(&attr, ptr) != hipSuccess || attr.type != hipMemoryTypeHost) {
        (void)hipGetLastError();
        return fail(c, HICR_EINVAL, "address is not pinned host memory");
      }
      void *dp = nullptr;
      if (hipHostGetDevicePointer(&dp, ptr, 0) != hipSuccess || !dp) {
        (void)hipGetLastError();
        return fail(c, HICR_EINVAL, "pinned host memory without a device address");
      }
      dev_addr = reinterpret_cast<uint64_t>(dp);
      void *last = static_cast<char *>(ptr) + (size - 1);
      void *dlast = nullptr;
      if (size > 1 && (hipHostGetDevicePointer(&dlast, last, 0) != hipSuccess ||
                       reinterpret_cast<uint64_t>(dlast) != dev_addr + (size - 1))) {
        (void)hipGetLastError();
        return fail(c, HICR_ERANGE, "slot extends past the end of its pinned allocation");
      }
    }
    if (c->slots.size() >= kMaxSlots)
      return fail(c, HICR_ENOMEM, "at most %u slots per context", kMaxSlots);
    Slot s;
    s.base = dev_addr;
    s.size = size;
    s.space = memspace;
    s.live = true;
    c->slots.push_back(s);
    *out = (hicr_slot)(c->slots.size() - 1);
    return HICR_OK;
  });
}

int hicr_slot_deregister(hicr_ctx c, hicr_slot slot) {
  return guarded([&]() -> int {
    if (!c) return HICR_EINVAL;
    std::lock_guard<std::mutex> g(c->mu);
    if (slot >= c->slots.size() || !c->slots[slot].live) return fail(c, HICR_EBADSLOT, "bad slot");
    for (const hicr_desc &d : c->pending)
      if (d.dst_slot == slot || d.src_slot == slot)
        return fail(c, HICR_EBUSY, "slot has unsubmitted transfers; fence first");
    if (c->slots[slot].plan_refs)
      return fail(c, HICR_EBUSY, "slot is used by %u plan(s)", c->slots[slot].plan_refs);
    if (c->slots[slot].dobj_refs)
      return fail(c, HICR_EBUSY, "slot holds %u published data object(s)", c->slots[slot].dobj_refs);
    (void)hipSetDevice(c->device);
    if (any_inflight(c) || extra_inflight(c) || plans_inflight(c))
      return fail(c, HICR_EBUSY, "transfers in flight; fence first");
    c->slots[slot].live = false;
    return HICR_OK;
  });
}

int hicr_slot_counters(hicr_ctx c, hicr_slot slot, uint64_t *sent, uint64_t *recv) {
  return guarded([&]() -> int {
    if (!c) return HICR_EINVAL;
    std::lock_guard<std::mutex> g(c->mu);
    if (slot >= c->slots.size() || !c->slots[slot].live) return fail(c, HICR_EBADSLOT, "bad slot");
    (void)hipSetDevice(c->device);
    // transfers counted in the slot, less those of submissions and replays
    // still in flight, plus what launches have counted on the device
    uint64_t n_sent = c->slots[slot].sent, n_recv = c->slots[slot].recv;
    (void)any_inflight(c);
    for (const Sub &s : c->subs) {
      if (!s.inflight) continue;
      const uint64_t *hp = static_cast<const uint64_t *>(s.h) + 3 * s.host_counted;
      for (uint64_t i = 0; i < s.host_counted; i++) {
        n_recv -= (hp[i] & 0xffffffffull) == slot;
        n_sent -= (hp[i] >> 32) == slot;
      }
    }
    plans_unfinished(c, slot, &n_sent, &n_recv);
    if (c->dev_counted) {
      hipError_t e = hipMemcpyAsync(c->h_read, c->d_counters + 2 * slot, 16, hipMemcpyDeviceToHost,
                                    c->aux);
      if (e == hipSuccess) e = hipStreamSynchronize(c->aux);
      if (e != hipSuccess) return hip_fail(c, e, "reading counters");
      n_sent += c->h_read[0];
      n_recv += c->h_read[1];
    }
    if (sent) *sent = n_sent;
    if (recv) *recv = n_recv;
    return HICR_OK;
  });
}

int hicr_memcpy(hicr_ctx c, hicr_slot dst, uint64_t dst_off, hicr_slot src, uint64_t src_off,
                uint64_t size) {
  return guarded([&]() -> int {
    if (!c) return HICR_EINVAL;
    std::lock_guard<std::mutex> g(c->mu);
    hicr_desc d{dst, src, dst_off, src_off, size};
    int rc = check_desc(c, d);
    if (rc != HICR_OK) return fail(c, rc, "memcpy rejected");
    c->pending.push_back(d);
    if (c->pending.size() >= kMaxLdsDescs) {
      (void)hipSetDevice(c->device);
      return flush_pending(c);
    }
    return HICR_OK;
  });
}

int hicr_memcpy_batch(hicr_ctx c, const hicr_desc *descs, uint64_t n, const hicr_sched *s,
                      void *stream, uint64_t *bad) {
  return guarded([&]() -> int {
    if (!c || (n && !descs)) return HICR_EINVAL;
    std::lock_guard<std::mutex> g(c->mu);
    (void)hipSetDevice(c->device);
    hicr_sched sched = s ? *s : c->def_sched;
    if (sched.mode == HICR_SCHED_TUNED || sched.mode == HICR_SCHED_LEARNED) {
      int rc = choose_sched(c, descs, n, sched.mode, &sched);
      if (rc != HICR_OK) return rc;
    } else if (sched.mode != HICR_SCHED_FIXED) {
      return fail(c, HICR_EINVAL, "unknown schedule mode %u", sched.mode);
    }
    int rc = check_sched(c, sched);
    if (rc != HICR_OK) return rc;
    rc = flush_pending(c);
    if (rc != HICR_OK) return rc;
    return submit(c, descs, n, sched,
                  stream ? static_cast<hipStream_t>(stream) : c->stream, bad, nullptr);
  });
}

int hicr_memcpy_batch_noalloc(hicr_ctx c, const hicr_desc *descs, uint64_t n, const hicr_sched *s,
                              void *stream, uint64_t *bad) {
  return guarded([&]() -> int {
    if (!c || (n && !descs)) return HICR_EINVAL;
    std::lock_guard<std::mutex> g(c->mu);
    if (n > kNoAllocMaxReqs)
      return fail(c, HICR_EINVAL, "%llu requests: the no-allocation path takes at most %llu",
                  (unsigned long long)n, (unsigned long long)kNoAllocMaxReqs);
    const hicr_sched sched = s ? *s : c->def_sched;
    if (sched.mode != HICR_SCHED_FIXED)
      return fail(c, HICR_EINVAL, "the no-allocation path takes a fixed schedule only");
    int rc = check_sched(c, sched);
    if (rc != HICR_OK) return rc;
    if (!c->na_scratch || !c->na_h) return fail(c, HICR_EDEVICE, "no device workspace");
    if (n == 0) return HICR_OK;
    (void)hipSetDevice(c->device);
    // the staging is reused: the previous call's upload must have finished
    if (c->na_up_pending) {
      hipError_t e = hipEventSynchronize(c->na_up_ev);
      if (e != hipSuccess) return hip_fail(c, e, "waiting for the previous upload");
      c->na_up_pending = false;
    }
    uint64_t *h = static_cast<uint64_t *>(c->na_h);
    const Packed k = pack_range(c, descs, n, 0, n, h);
    if (k.rc != HICR_OK) {
      if (bad) *bad = k.bad;
      return fail(c, k.rc, "request %llu rejected", (unsigned long long)k.bad);
    }
    if (k.bytes >= kNoAllocMaxBytes)
      return fail(c, HICR_EINVAL, "%llu bytes: the no-allocation path moves less than 2^38 per call",
                  (unsigned long long)k.bytes);
    const DevSched ds{sched.chunk_bytes, sched.wgs_per_desc, sched.unroll, 0};
    rc = split_batch(c, h, h + 2 * n, n, ds, c->segs);
    if (rc != HICR_OK) return rc;
    const hipStream_t st = stream ? static_cast<hipStream_t>(stream) : c->stream;
    // upload, scans, copies and counters all run in order on one stream; a
    // previous call of this context on another stream must have left the
    // workspace first
    hipError_t e = hipSuccess;
    if (c->na_inflight) e = hipStreamWaitEvent(st, c->na_ev, 0);
    if (e == hipSuccess) e = hipMemcpyAsync(c->na_scratch, h, n * 32, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipEventRecord(c->na_up_ev, st);
    if (e != hipSuccess) return hip_fail(c, e, "uploading a batch");
    c->na_up_pending = true;
    const uint64_t *dd = static_cast<const uint64_t *>(c->na_scratch);
    uint32_t *tables = batch_tables(c->na_scratch, n);
    c->dev_counted = true;
    rc = launch_scans(c, nullptr, dd, n, c->segs, ds, tables, st);
    if (rc == HICR_OK) rc = launch_copies(c, dd, n, c->segs, ds, tables, c->d_counters, st);
    e = hipEventRecord(c->na_ev, st);
    if (e == hipSuccess) c->na_inflight = true;
    if (rc != HICR_OK) return rc;
    if (e != hipSuccess) return hip_fail(c, e, "recording a batch event");
    return HICR_OK;
  });
}

int hicr_fence(hicr_ctx c) {
  return guarded([&]() -> int {
    if (!c) return HICR_EINVAL;
    std::lock_guard<std::mutex> g(c->mu);
    (void)hipSetDevice(c->device);
    int rc = flush_pending(c);
    int r2 = wait_all(c);
    return rc != HICR_OK ? rc : r2;
  });
}

int hicr_fence_slot(hicr_ctx c, hicr_slot slot, uint64_t exp_sent, uint64_t exp_recv,
                    uint64_t timeout_ns) {
  return guarded([&]() -> int {
    if (!c) return HICR_EINVAL;
    {
      std::lock_guard<std::mutex> g(c->mu);
      if (slot >= c->slots.size() || !c->slots[slot].live) return fail(c, HICR_EBADSLOT, "bad slot");
      (void)hipSetDevice(c->device);
      int rc = flush_pending(c);
      if (rc != HICR_OK) return rc;
    }
    auto t0 = std::chrono::steady_clock::now();
    for (;;) {
      bool busy;
      {
        std::lock_guard<std::mutex> g(c->mu);
        busy = any_inflight(c) || extra_inflight(c) || plans_inflight(c);
      }
      uint64_t s = 0, r = 0;
      int rc = hicr_slot_counters(c, slot, &s, &r);
      if (rc != HICR_OK) return rc;
      if (s >= exp_sent && r >= exp_recv) return HICR_OK;
      if (!busy) return fail(c, HICR_ETIMEDOUT, "expected counts cannot be reached");
      auto dt = std::chrono::duration_cast<std::chrono::nanoseconds>(
                    std::chrono::steady_clock::now() - t0).count();
      if ((uint64_t)dt >= timeout_ns) return fail(c, HICR_ETIMEDOUT, "fence_slot timed out");
      std::this_thread::sleep_for(std::chrono::microseconds(20));
    }
  });
}

}  // extern "C"
