// runtime.h -- the host context shared by the runtime's translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <map>
#include <mutex>
#include <string>
#include <unordered_set>
#include <vector>

#include "hicr.h"
#include "internal.h"

struct hicr_channel_s;
struct hicr_plan_s;

namespace hicr {

struct Slot {
  uint64_t base = 0;
  uint64_t size = 0;
  uint32_t space = 0;
  uint32_t plan_refs = 0;  // plans whose requests name this slot
  uint32_t dobj_refs = 0;  // published data objects inside this slot
  bool live = false;
  // transfers accepted by submissions whose end the host sees itself (Done):
  // the slot's counters are these, less what is still in flight, plus the
  // device's
  uint64_t sent = 0, recv = 0;
  uint64_t tmp_sent = 0, tmp_recv = 0;  // while a plan is made: its transfers of this slot
};

// The words of pinned host memory a launch raises when it ends (Done), and
// the launch's event.  On the context's own stream the event is recorded only
// once somebody has to wait for it: recording one after every launch cost
// the stream ~8 us each, and nobody else can queue work there behind the
// library's.
struct Signal {
  uint64_t *words = nullptr;  // kDoneWords of them
  uint32_t *arrive = nullptr;
  uint64_t seq = 0;           // value of the last launch's words
  uint32_t n_words = 0;       // words the last launch raises (0: only the event tells)
  hipEvent_t ev = nullptr;
  bool recorded = false;      // ev has been recorded behind the last launch
};

// One submission buffer: pinned staging, its device copy, and how the
// submission's end is seen.
struct Sub {
  void *h = nullptr;      // staging (the context's own block up to kStageReqs requests)
  void *h_dev = nullptr;  // its device address
  void *d = nullptr;
  uint64_t h_cap = 0, d_cap = 0;  // requests they have room for
  hipEvent_t up_ev = nullptr;  // end of its upload, when that ran on the upload stream
  Signal sig;
  bool inflight = false;
  uint64_t host_counted = 0;   // its first requests counted in the slots (all, or none)
  uint64_t push_seq = 0;       // host-API pushes and network steps queued before it on its stream
};

class HostPool;  // host threads that validate and pack large batches (runtime.cpp)

// One copy launch of a batch: requests [i0, i1) with `bytes` bytes and
// `pieces` pieces (exact on the LDS path, at least that many on the table
// path); `lds` when every workgroup scans the piece table into LDS itself,
// otherwise the launch reads the tables that scan_kernel wrote.
struct Seg {
  uint64_t i0, i1, pieces, bytes;
  bool lds;
};

// Extra controls of one submission (autotuner).
struct SubmitOpts {
  bool no_count = false;     // do not raise slot counters
  hipEvent_t t0 = nullptr;   // recorded just before the first scan or copy launch
  hipEvent_t t1 = nullptr;   // recorded just after the last copy launch
};

constexpr int kNumSubs = 4;
constexpr uint64_t kStageReqs = 1024;   // staged by a submission buffer from the start
// Staging of n requests: 32 bytes each, then the stream kernel's starts.
constexpr size_t stage_bytes(uint64_t n) {
  return (n * 32 + (kMaxStreamWaves + 1) * sizeof(StreamStart) + 4095) & ~(size_t)4095;
}
constexpr uint32_t kMaxSlots = 1u << 20;  // slots per context (fixed counter table)

struct SchedState;  // autotuned table and device-resident network (sched.cpp)

// Asynchronous work other than copy submissions (channel pushes, pumps):
// its event, and buffers to free once it has completed.
// Staging (pinned) and device buffers of a pump launch, reused by later
// launches once the pump has finished: allocating and freeing them per call
// cost ~1 ms, and hipFree waits for the device.
struct PumpBuf {
  void *h = nullptr, *d = nullptr;
  uint64_t h_cap = 0, d_cap = 0;
};

// A pump launch whose completion has not been observed yet: what later
// launches need to stay co-resident with it and off its rings.
struct PumpLive {
  hipEvent_t ev = nullptr;
  hipStream_t stream = nullptr;
  uint64_t wgs = 0;
  std::vector<struct ::hicr_channel_s *> chans;
};

struct Extra {
  hipEvent_t ev = nullptr;
  void *d_buf = nullptr;
  void *h_buf = nullptr;
  uint64_t h_cap = 0, d_cap = 0;  // sizes of h_buf and d_buf
  bool pump = false;
  uint32_t *abort_word = nullptr;
  std::vector<struct ::hicr_channel_s *> chans;
};

}  // namespace hicr

struct hicr_ctx_s {
  std::mutex mu;
  int device = 0;
  hipStream_t stream = nullptr;
  bool own_stream = false;
  hipStream_t aux = nullptr;  // counter reads, never waits on `stream`
  hipStream_t up = nullptr;   // uploads of large batches, overlapping earlier copies
  hicr::HostPool *pool = nullptr;  // created at the first large submission
  bool pool_failed = false;        // its threads could not be started
  int n_cu = 1;
  int occ = 1;       // copy workgroups per CU that fit
  int grid_per_cu = 0;  // copy workgroups per CU launched (0: per-schedule default)
  uint32_t pair_mask = HICR_PAIRS_ALL;  // memory-space pairs memcpy accepts
  std::vector<hicr::Slot> slots;
  uint64_t *d_counters = nullptr;  // [slot] = {sent, recv}
  uint32_t counter_cap = 0;
  uint64_t *h_read = nullptr;  // pinned read-back buffer
  hicr::Sub subs[hicr::kNumSubs];
  int next_sub = 0;
  uint64_t *h_done = nullptr;    // the submission buffers' done words; heads the context's pinned block
  bool dev_counted = false;      // some launch has counted its requests on the device
  // hicr_memcpy_batch_noalloc: this device's fixed workspace, pinned staging
  // allocated with the context, and the events of the last such submission
  void *na_scratch = nullptr;
  void *na_h = nullptr;
  hipEvent_t na_up_ev = nullptr;  // end of its upload (the staging is free again)
  hipEvent_t na_ev = nullptr;     // end of its last launch
  bool na_up_pending = false;
  bool na_inflight = false;
  std::vector<hicr::Seg> segs;  // launches of the submission being queued
  std::vector<hicr_desc> pending;
  hicr_sched def_sched{};
  hicr::SchedState *sched = nullptr;
  std::unordered_set<struct hicr_channel_s *> channels;
  std::vector<struct hicr_plan_s *> plans;
  std::vector<void *> plan_blocks;      // pinned blocks of plans' done words,
  std::vector<uint64_t *> plan_words;   // and the words in them that are free
  std::map<uint64_t, hicr_dobj_handle> dobjs;  // published data objects by id
  uint64_t next_dobj_id = 1;
  std::vector<hicr::Extra> extra;
  std::vector<hicr::PumpBuf> pump_free;  // finished pumps' buffers, for reuse
  std::vector<hicr::PumpLive> pump_live;  // pumps launched and not yet finished
  int pump_occ = 0;  // pump workgroups per CU
  std::vector<hipStream_t> serve_streams;  // of hicr_serve, kept for its next call
  // host-API channel pushes and network steps queued on `stream`: how many,
  // how many of them are known to have ended, and the event of the last
  uint64_t push_seq = 0, push_done = 0;
  hicr::Signal push_sig;
  // words of hicr_pingpong launches and their copy on the host (pinned)
  uint64_t *pp_d = nullptr, *pp_h = nullptr;
  size_t pp_words = 0;
  std::mutex abort_mu;  // guards abort_words; never held while waiting on the GPU
  std::vector<uint32_t *> abort_words;  // running pumps' pinned abort words
  std::string err;
};

namespace hicr {

int fail(hicr_ctx c, int code, const char *fmt, ...);
int hip_fail(hicr_ctx c, hipError_t e, const char *what);
int check_desc(hicr_ctx c, const hicr_desc &d);
int check_sched(hicr_ctx c, const hicr_sched &s);
bool any_inflight(hicr_ctx c);
// Wait for an event: poll briefly, then block.
hipError_t sync_event(hipEvent_t e);
// The next launch of `grid` workgroups raises sig's words.
inline Done arm(Signal &sig, uint32_t grid) {
  sig.n_words = done_words(grid);
  return Done{sig.words, sig.arrive, ++sig.seq};
}
// Queue what marks the end of everything launched on `s` so far: the event,
// unless `s` is the context's own stream.
hipError_t mark(hicr_ctx c, Signal &sig, hipStream_t s);
// Whether the marked launch has ended / wait until it has (its words are
// polled for up to 200 us, then the event is waited for).
bool ended(hicr_ctx c, Signal &sig);
hipError_t wait_signal(hicr_ctx c, Signal &sig);
// The event behind the marked launch, recorded now if it is not yet.
hipError_t ensure_event(hicr_ctx c, Signal &sig);
// Whether a caller is capturing stream s into a graph.
bool capturing(hicr_ctx c, hipStream_t s);
// Whether every request of a batch writes device memory (HBM slots): only
// then may done words stand for the end of the batch, since the runtime's
// completion signal is what makes bytes written to host memory visible.
bool writes_device_only(hicr_ctx c, const hicr_desc *d, uint64_t n);
int wait_all(hicr_ctx c);
int submit(hicr_ctx c, const hicr_desc *d, uint64_t n, const hicr_sched &sched,
           hipStream_t stream, uint64_t *bad, const SubmitOpts *opt);
int flush_pending(hicr_ctx c);
// Resolve requests to the structure of arrays {dst, src, size, slot pair}.
void pack_batch(hicr_ctx c, const hicr_desc *d, uint64_t n, uint64_t *h);
// Split an n-request batch into copy launches (hd/hz: host copies of dst and
// size): one LDS-scanned launch up to kMaxLdsDescs requests, otherwise
// launches over a scanned table of at most kTile * kMaxTiles requests; every
// launch under 2^31 pieces.
int split_batch(hicr_ctx c, const uint64_t *hd, const uint64_t *hz, uint64_t n, const DevSched &ds,
                std::vector<Seg> &out);
// Queue the scan kernel for every launch that reads a table (tables: the
// batch_tables() region beside the batch dd).  staged: the batch lies there,
// in pinned host memory, and the kernel moves it to dd.
int launch_scans(hicr_ctx c, const uint64_t *staged, const uint64_t *dd, uint64_t n, 
                 const std::vector<Seg> &segs, DevSched ds, uint32_t *tables, hipStream_t stream);
// Queue the copy launches, then (counters != null) the counter kernel.  With
// sig != null and a single copy launch, that launch raises sig's words.
int launch_copies(hicr_ctx c, const uint64_t *dd, uint64_t n, const std::vector<Seg> &segs,
                  DevSched ds, const uint32_t *tables, uint64_t *counters, hipStream_t stream,
                  Signal *sig = nullptr);
// Queue the counter kernel over the slot pairs of a batch dd (counters null: none).
int launch_counts(hicr_ctx c, const uint64_t *dd, uint64_t n, uint64_t *counters,
                  hipStream_t stream, Signal *sig);
// Bytes of device memory an uploaded batch of n requests takes: the packed
// requests (32 B each), then the piece tables: per-request prefixes (4 B
// each) and tile totals (a launch over requests [i0, i1) keeps its tiles at
// entry i0 of an n-entry region; it has fewer tiles than requests).
inline uint64_t batch_bytes(uint64_t n) { return n * 40; }
inline uint32_t *batch_tables(void *d, uint64_t n) {
  return reinterpret_cast<uint32_t *>(static_cast<char *>(d) + n * 32);
}

// Persistent batch plans (plan.cpp).
int wait_plans(hicr_ctx c);
bool plans_inflight(hicr_ctx c);
void destroy_plans(hicr_ctx c);
// Take what the plans' replays in flight will count on `slot` off the counts.
void plans_unfinished(hicr_ctx c, uint32_t slot, uint64_t *sent, uint64_t *recv);

// Schedule selection (sched.cpp): the class for a batch under mode TUNED
// (nearest tuned-table entry) or LEARNED (the network: on the host, in the
// device kernels' arithmetic, per submission; by the device forward kernel
// when on_device, as for a plan's one-time choice); the context default when
// neither has data, or when no class would change how the batch is copied
// (unless pieces: the piece kernels take it whatever its size) and the table
// would be searched for nothing.  The network is asked in any case
// (hicr_last_choice).
int choose_sched(hicr_ctx c, const hicr_desc *d, uint64_t n, uint32_t mode, hicr_sched *out,
                 bool on_device = false, bool pieces = false);
// Whether a batch (not checked yet) is copied as one stream under every schedule.
bool same_under_every_class(hicr_ctx c, const hicr_desc *d, uint64_t n);
void destroy_sched(hicr_ctx c);

// Channel pushes and pumps (channel.cpp).
struct PumpStream {
  struct ::hicr_channel_s *channel;
  uint32_t producer;
  uint64_t src_base, src_size, out_base, out_size;
  uint64_t first_msg, n_msgs;
};
// msg_off/msg_size: host arrays, or (dev_tables) device arrays the kernel
// reads in place and checks itself.
int pump_launch(hicr_ctx c, const std::vector<PumpStream> &st, const uint64_t *msg_off,
                const uint64_t *msg_size, uint64_t n_msgs, uint32_t *trace_dev, uint64_t *ts_dev,
                uint64_t timeout_ns, hipStream_t s, Extra *xout, bool dev_tables = false);
int pump_finish(hicr_ctx c, Extra &x);
void destroy_pump_bufs(hicr_ctx c);
uint64_t channel_payload_limit(struct ::hicr_channel_s *ch);
int wait_extra(hicr_ctx c);
bool extra_inflight(hicr_ctx c);
void destroy_extra(hicr_ctx c);

// Every C entry point runs its body through guarded(): the ABI never throws.
// The only exceptions host code here can raise come from allocation (a
// container growing, new, a thread that cannot start), so each becomes
// HICR_ENOMEM; locks taken in the body are released on the way out.
template <class F>
inline int guarded(F &&body) noexcept {
  try {
    return body();
  } catch (...) {
    return HICR_ENOMEM;
  }
}

}  // namespace hicr
