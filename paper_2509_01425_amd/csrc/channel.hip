// channel.hip -- gfx950 kernels of the ring channels (HiCR Sec. 4.3).
//
// Protocol (per ring; counters monotone, see chan.h):
//   producer: wait until the consumer's released counters leave room for the
//             message (entries tm - hm < E, bytes tb - hb + s <= P), write the
//             payload at byte position tb mod P (split across the ring end),
//             write the entry, wait until those writes have reached the
//             device's coherence point, publish tm + 1;
//   consumer: read tm; while tm > hm read entry hm mod E and the payload at
//             hb mod P, then publish hb + s and hm + 1 -- the notification
//             that frees the producer's room.
// Locking MPSC: a ticket lock (FIFO-fair) guards the room check and the
// reservation of [rb, rb + s) / entry rm, which are handed on with the turn; the copy runs outside the lock and
// publication follows ticket order, so the shared ring holds one total order
// and never overflows.  Non-locking MPSC: one ring per producer.
//
// Everything that two workgroups exchange inside one pump -- payload, entries,
// records, counters -- moves with agent-scope accesses (cache bit sc1: loads
// miss the caches that are not coherent across XCDs, stores write through
// them), so no fence is needed beside them: a producer's writes are visible
// device-wide once its wave has waited for them (s_waitcnt vmcnt(0)), and a
// consumer may free room once its loads have returned.  An agent-scope
// release fence writes back the whole L2 of its XCD and an acquire
// invalidates it; with one of each per batch those write-backs bounded the
// pump (1,536 streams, 500 K messages of 16 B - 64 KiB: 6.28 ms with the
// fences and plain payload accesses, 2.8 ms now = 5.6 TB/s of source, ring
// and output bytes, what a large copy reaches; 1,024 SPSC streams and 64
// locking rings, 150 K messages to 256 KiB: 7.6 ms, 3.1 ms now = 5.2 TB/s).
//
// pump_kernel is persistent: an endpoint (the producer of one stream, the
// consumer of one or more single-producer rings) is either one wave, four of
// them to a workgroup, or a whole workgroup when the device holds one for
// every endpoint (few streams: the copy rate of one wave would bound each), or
// several workgroups while there are compute units to spare.
// Either way its messages are cut into chunks of kChunkRows KiB that the
// endpoint's waves take in turn, with the next chunk's loads issued before
// the current chunk's stores.  A single-producer ring's messages lie back to
// back in the ring and in the output, so its consumer copies everything it
// takes as one range.  The host launches no more workgroups than the device
// holds at once, and every wait gives up after a no-progress time-out or on
// the abort word, so every wave exits.
#include "chan.h"
#include "internal.h"
#include "span.h"

namespace hicr {

__device__ __forceinline__ uint64_t ld_rlx(uint64_t a) {
  return __hip_atomic_load((uint64_t *)a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_rlx(uint64_t a, uint64_t v) {
  __hip_atomic_store((uint64_t *)a, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// No-progress watchdog for spin waits.
// The error and abort words are shared by every wave of the pump, so a wave
// looks at them at most once per kWatchTicks of its own waiting (10 us of the
// 100 MHz clock) instead of on every poll: thousands of spinning waves
// reading one address would otherwise queue at one memory channel.  The
// host asks for an abort in pinned host memory (a plain store, so that no
// queue has to run beside the pump; err[4..5] hold that word's address): a
// wave reads it over the host link only in one of every 1,024 windows of
// 1,024 ticks (about once per 10 ms of its own waiting), the windows
// staggered over the waves so that their reads do not arrive together and
// a pump with many waiting waves sees the request within tens of
// microseconds, and passes a request on to err[1], which every wave reads.
// (Measured on the channel workload: reading it in one window of 128, all
// waves in the same one, cost 3 % of the pump's rate; one of 1,024, 0.3-1 %.)
constexpr uint64_t kWatchTicks = 1000;

// An error goes into the device's word, which every waiting wave looks at,
// and into one of the host's own words beside its abort word (one per kind:
// nothing has to be read back behind the pump: one of five streams 34 -> 32 us).
__device__ __forceinline__ void tell_host(uint32_t *err, uint32_t bit) {
  uint32_t *host = reinterpret_cast<uint32_t *>(__hip_atomic_load(
      reinterpret_cast<uint64_t *>(err + 4), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  if (host)
    __hip_atomic_store(host + kHostErrors + bit, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ void raise_error(uint32_t *err, uint32_t bit) {
  __hip_atomic_fetch_or(&err[0], bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  tell_host(err, bit);
}

struct Watch {
  uint64_t deadline, span;
  uint32_t *err;
  uint64_t next;
  __device__ void progress() { deadline = wall_clock64() + span; }
  // true when the wait must stop (time-out recorded, or abort requested)
  __device__ bool expired() {
    const uint64_t now = wall_clock64();
    if (now < next) return false;
    next = now + kWatchTicks;
    const uint32_t salt = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if ((((now >> 10) + salt) & 1023) == 0) {
      const uint32_t *host = reinterpret_cast<const uint32_t *>(__hip_atomic_load(
          reinterpret_cast<uint64_t *>(err + 4), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
      if (host && __hip_atomic_load(host, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM)) {
        if (__lane_id() == 0) {
          __hip_atomic_store(&err[1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          tell_host(err, kErrAbort);
        }
        return true;
      }
    }
    if (__hip_atomic_load(&err[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ||
        __hip_atomic_load(&err[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      return true;
    if (now > deadline) {
      raise_error(err, kErrTimeout);
      return true;
    }
    return false;
  }
  // The same for a wait that outlasts many steps of others (an end of a split
  // ring: its next share may lie far down the stream): a change of what it
  // polls is progress, and so is its first look.
  uint64_t seen;
  __device__ void poll() { seen = ~0ull; }
  __device__ bool stuck(uint64_t v) {
    if (v == seen) return expired();
    seen = v;
    progress();
    return false;
  }
};

__device__ __forceinline__ uint64_t shfl64(uint64_t v, int src) {
  return ((uint64_t)__shfl((unsigned)(v >> 32), src) << 32) | (uint64_t)__shfl((unsigned)v, src);
}

// A table entry that nothing writes while the kernel runs, at an index that
// is the same in every lane: read through the scalar cache into scalar
// registers (the compiler does so by itself only before the first store).
template <class T>
__device__ __forceinline__ T table(const T *p) {
  static_assert(sizeof(T) % 4 == 0, "whole words");
  const __attribute__((address_space(4))) uint32_t *w =
      (const __attribute__((address_space(4))) uint32_t *)uni64((uint64_t)p);
  uint32_t t[sizeof(T) / 4];
#pragma unroll
  for (uint32_t i = 0; i < sizeof(T) / 4; i++) t[i] = w[i];
  T v;
  __builtin_memcpy(&v, t, sizeof(T));
  return v;
}

// Inclusive prefix sum over the 64 lanes of a wave.
__device__ __forceinline__ uint64_t wave_scan(uint64_t v, uint32_t lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    uint64_t t = ((uint64_t)__shfl_up((unsigned)(v >> 32), o) << 32) | __shfl_up((unsigned)v, o);
    if (lane >= (uint32_t)o) v += t;
  }
  return v;
}

// Store two words of one 16-byte unit with one access (lanes outside `on`
// store nothing), so that whoever reads the first also finds the second.
__device__ __forceinline__ void st_pair(uint64_t a, uint64_t w0, uint64_t w1, bool on) {
  v4i v;
  v.x = (int32_t)w0;
  v.y = (int32_t)(w0 >> 32);
  v.z = (int32_t)w1;
  v.w = (int32_t)(w1 >> 32);
  bstore<16>(span_rsrc(a, 16), on ? 0u : ~0u, v);
}

// Read such a unit with one access, the same in every lane.
__device__ __forceinline__ v4i ld_pair(uint64_t a) { return bload<16>(span_rsrc(a, 16), 0); }
__device__ __forceinline__ uint64_t lo64(v4i v) {
  return (uint32_t)v.x | (uint64_t)(uint32_t)v.y << 32;
}
__device__ __forceinline__ uint64_t hi64(v4i v) {
  return (uint32_t)v.z | (uint64_t)(uint32_t)v.w << 32;
}

// Ring bytes are written without nt: the consumer reads most of them soon
// after, and they then come from the memory-side cache (4.03 against 4.42 ms
// a pass on the first configuration above; reading the ring without nt
// 4.3-4.4 ms).

// Messages l to j - 1 between a ring and other memory, as a sequence of
// chunks: lane l holds message l's size, ring position (below P) and other
// address.  Chunks end at destination line boundaries, message ends and the
// ring end.
template <bool kToRing>
struct Feed {
  uint64_t payload, P;
  uint64_t v_size, v_pos, v_addr;
  uint32_t j, l = 0;
  uint64_t left = 0, pos = 0, addr = 0;
  __device__ __forceinline__ Chunk next() {
    while (left == 0 && l < j) {
      left = lane64(v_size, l);
      pos = lane64(v_pos, l);
      addr = lane64(v_addr, l);
      l++;
    }
    Chunk c;
    const uint64_t ring = payload + pos;
    c.d = kToRing ? ring : addr;
    c.s = kToRing ? addr : ring;
    uint64_t n = kChunkBytes - (c.d & (kLineBytes - 1));
    if (n > left) n = left;
    if (n > P - pos) n = P - pos;
    c.n = __builtin_amdgcn_readfirstlane((uint32_t)n);
    left -= n;
    addr += n;
    pos += n;
    if (pos == P) pos = 0;
    return c;
  }
  __device__ __forceinline__ void skip(uint32_t k) {
    for (uint32_t i = 0; i < k; i++) (void)next();
  }
};

// Move the messages of a feed with an endpoint of WAVES waves: wave w takes
// chunks w, w + WAVES, ...  On return every load has completed; stores may
// still be in flight.
template <int WAVES, bool kToRing>
__device__ __forceinline__ void move_feed(Feed<kToRing> f, uint32_t wave, uint32_t lane) {
  if (WAVES > 1) f.skip(wave);
  move_chunks<kToRing ? kReadStream : kAgentStream, kToRing ? kAgent : kAgentStream>(
      [&]() {
        const Chunk c = f.next();
        if (WAVES > 1) f.skip(WAVES - 1);
        return c;
      },
      lane);
}

// What the first wave of a workgroup endpoint tells the others per batch.
struct Cast {
  uint64_t w[4];
  uint32_t stop, late_stop;
};

// Messages a producer publishes at once.  On a locking ring a batch also ends
// at an eighth of the ring's bytes (unless its first message is larger), and
// so does a round of the consumer team: the ring holds several batches and
// rounds at different stages at once, where one of half the ring made the
// others wait (64 rings, 8 producers each, messages to 256 KiB: 1.80 ms with
// the eighths, 2.15 ms without; with 1,024 SPSC streams beside them 4.84
// against 5.1 ms a pass; a sixteenth 1.84, a quarter 1.83).
constexpr uint32_t kProdBatch = 16;
constexpr uint32_t kLockShare = 8;

// Who goes first.  Beside 1,024 SPSC streams the locking rings, which move
// their bytes in ordered steps, were left for last (their ends 2.6-3.6 ms into
// a pass of 3.84 ms, the others' 1.1-3.3): their waves now have priority in
// their SIMD, consumers (3) over producers (2): 3.54 ms; and so have the
// consumers of other rings (1) over the producers (0), which keeps what a ring
// holds nearer to its use: 3.42 ms, and without locking rings 3.03 -> 2.98.
// A single wave also starts no message while its ring is filled to more than
// a quarter (or kWaveFill bytes), which gives way to the locking rings without
// keeping its consumer waiting: 3.27 ms.  (A half 3.33; with rings of 256 KiB
// a quarter made 900 streams 4 % slower, kWaveFill nothing; whole workgroups
// drain their rings fast enough as it is, 300 streams 1,130 -> 1,320 us.)
// Giving the larger streams priority over the smaller made a pass 2 % slower.
constexpr uint64_t kWaveFill = 128 << 10;

// The producer of one stream (WAVES waves): it takes as many of its next
// messages as the ring has room for, copies them as one batch and writes
// their entries.  A batch is published at the top of the next turn, after
// one wait that covers its stores and the loads of the next messages' sizes.
template <int WAVES>
__device__ void run_producer(const PumpArgs &a, uint32_t sid_in, uint32_t wave, uint32_t lane,
                             Cast *cast) {
  // the stream id is the same in every lane of the wave; saying so lets the
  // stream and ring descriptors live in scalar registers
  const uint32_t sid = __builtin_amdgcn_readfirstlane(sid_in);
  const DevStream st = table(&a.streams[sid]);
  const DevRing r = table(&a.rings[st.ring]);
  const bool locking = table(&a.chans[st.channel].mode) == kModeMpscLock;
  const uint64_t fill = locking || WAVES > 1 ? r.P : r.P / 4 > kWaveFill ? r.P / 4 : kWaveFill;
  if (locking) __builtin_amdgcn_s_setprio(2);
  const uint64_t c = r.coord;
  const uint64_t tm_a = c + offsetof(RingCoord, prod), hm_a = c + offsetof(RingCoord, cons),
                 hb_a = hm_a + 8, tk_a = c + offsetof(RingCoord, lock), tn_a = tk_a + 16;
  // rings are empty when a pump starts: the producer side resumes at the
  // consumer's released counters
  uint64_t tm = uni64(ld_rlx(tm_a)), tb = uni64(ld_rlx(hb_a));
  Watch w{0, a.timeout_ticks, a.err, 0, 0};
  w.progress();
  uint64_t m = 0;
  uint64_t out_run = 0;  // output bytes of this stream's earlier messages
  uint32_t last_j = 0;   // messages of the batch not yet published
  for (;;) {
    // sizes and offsets of the next messages, one per lane
    const bool have = lane < kProdBatch && m + lane < st.n_msgs;
    const uint64_t sz = have ? a.msg_size[st.first_msg + m + lane] : 0;
    const uint64_t off = have ? a.msg_off[st.first_msg + m + lane] : 0;
    drain();
    if (WAVES > 1) __syncthreads();
    bool stop = false;
    if (wave == 0 && last_j) {
      // the previous batch's payload and entries are in place: publish it, on
      // a locking ring in reservation order
      if (locking)
        while (uni64(ld_rlx(tm_a)) != tm - last_j) {
          __builtin_amdgcn_s_sleep(1);
          if (w.expired()) {
            stop = true;
            break;
          }
        }
      if (!stop) {
        if (a.ts_push && lane < last_j) a.ts_push[st.first_msg + m - last_j + lane] = wall_clock64();
        if (lane == 0) {
          // a ring of its own also publishes its byte counter, the form user
          // kernels (hicr_device.h) resume from
          if (!locking) st_rlx(tm_a + 8, tb);
          st_rlx(tm_a, tm);
        }
      }
      w.progress();
    }
    const uint64_t incl = wave_scan(sz, lane);
    // every message is checked before a byte of it moves (the host has not
    // seen message tables that live on the device): it fits the ring, its
    // source range lies in the stream's source slot, its output in the
    // output slot
    const bool bad = have && (sz > r.P || off > st.src_bytes || sz > st.src_bytes - off ||
                              out_run + incl > st.out_bytes);
    if (m >= st.n_msgs) return;
    if (__ballot(bad)) {
      if (wave == 0 && lane == 0)
        raise_error(a.err, kErrCorrupt);
      return;
    }
    uint64_t my_tm = tm, my_tb = tb, hm = 0, hb = 0, ticket = 0;
    if (wave == 0) {
      if (locking && !stop) {
        if (lane == 0)
          ticket = __hip_atomic_fetch_add((uint64_t *)tk_a, 1ull, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
        ticket = shfl64(ticket, 0);
        // the turn comes with the reservation counters in one 16-byte unit: a
        // lock handed over by one store and taken with one read (one ring of
        // 8 producers 1,850 us with a word each, 1,810 so; reading the
        // consumer's counters in the same loop 2,010: more to poll)
        for (;;) {
          order();
          const v4i turn = ld_pair(tn_a);
          if (uni64(lo64(turn)) << 32 == ticket << 32) {
            my_tm = r.base_m + (uint32_t)((uint32_t)(uni64(lo64(turn)) >> 32) - (uint32_t)r.base_m);
            my_tb = uni64(hi64(turn));
            break;
          }
          __builtin_amdgcn_s_sleep(1);
          if (w.expired()) {
            stop = true;
            break;
          }
        }
        order();
      }
      // wait until at least the first message fits, then take every leading
      // message that fits in the room seen (one view of the consumer for the
      // whole endpoint)
      const uint64_t s0 = shfl64(sz, 0);
      while (!stop) {
        hm = uni64(ld_rlx(hm_a));
        hb = uni64(ld_rlx(hb_a));
        if (my_tm - hm < r.E && my_tb - hb <= fill && my_tb - hb + s0 <= r.P) break;
        __builtin_amdgcn_s_sleep(2);
        if (w.expired()) stop = true;
      }
      order();
    }
    if (WAVES > 1) {
      if (wave == 0 && lane == 0) {
        cast->w[0] = my_tm;
        cast->w[1] = my_tb;
        cast->w[2] = hm;
        cast->w[3] = hb;
        cast->stop = stop;
      }
      __syncthreads();
      my_tm = cast->w[0];
      my_tb = cast->w[1];
      hm = cast->w[2];
      hb = cast->w[3];
      stop = cast->stop;
    }
    if (stop) return;
    const bool fits = have && (my_tm + lane + 1 - hm <= r.E) && (my_tb + incl - hb <= r.P) &&
                      my_tb + incl - sz - hb <= fill &&
                      (!locking || lane == 0 || incl <= r.P / kLockShare);
    const uint64_t fm = __ballot(fits);
    const uint32_t j = (uint32_t)__ffsll((unsigned long long)~fm) - 1;  // leading fitting lanes
    const uint64_t bytes = shfl64(incl, (int)j - 1);
    if (locking && wave == 0)
      st_pair(tn_a, (uint32_t)(ticket + 1) | (my_tm + j) << 32, my_tb + bytes, lane == 0);
    // entries (and, on a locking ring, the records the consumer team reads)
    // are written now; the wait before publication covers them
    if (wave == 0 && lane < j) {
      st_rlx(r.entries + 8 * ((my_tm + lane) % r.E), sz | ((uint64_t)st.producer << 48));
      if (locking) {
        // the message's record for the consumer team: ring byte position,
        // output address, message index (a counter outside this pump's
        // records means the ring's state is not what the host planned for)
        const uint64_t idx = my_tm + lane - r.base_m;
        if (idx < r.side_n) {
          const uint64_t rec = r.side + 24 * idx;
          st_rlx(rec, my_tb + incl - sz);
          st_rlx(rec + 8, st.out_base + out_run + incl - sz);
          st_rlx(rec + 16, st.first_msg + m + lane);
        } else {
          raise_error(a.err, kErrCorrupt);
        }
      }
    }
    Feed<true> f;
    f.payload = r.payload;
    f.P = r.P;
    f.v_size = sz;
    f.v_pos = (my_tb + incl - sz) % r.P;
    f.v_addr = st.src_base + off;
    f.j = j;
    move_feed<WAVES, true>(f, wave, lane);
    tm = my_tm + j;
    tb = my_tb + bytes;
    m += j;
    out_run += bytes;
    last_j = j;
    w.progress();
  }
}

// The consumer of a set of independent rings (WAVES waves), each with a
// single producer stream (SPSC rings, non-locking MPSC sub-rings): lane q
// keeps ring q's state.  Each turn takes up to 64 published messages of one
// ring (round robin over the rings that have any), at most a quarter of the
// ring's bytes unless the first message is larger, so that the producer gets
// room back while the rest is copied; copies them as one range to their
// stream's output and releases their room.
template <int WAVES>
__device__ void run_consumer(const PumpArgs &a, uint32_t uid_in, uint32_t wave, uint32_t lane,
                             Cast *cast) {
  const uint32_t uid = __builtin_amdgcn_readfirstlane(uid_in);
  const DevChannel u = table(&a.chans[uid]);
  __builtin_amdgcn_s_setprio(1);
  const bool mine = lane < u.n_rings;
  uint64_t coord = 0, hm = 0, hb = 0, pos = 0, out_pos = 0, cnt = 0;
  if (mine) {
    const DevRing rg = a.rings[u.first_ring + lane];
    coord = rg.coord;
    hm = ld_rlx(coord + offsetof(RingCoord, cons));
    hb = ld_rlx(coord + offsetof(RingCoord, cons) + 8);
    pos = hb % rg.P;
  }
  Watch w{0, a.timeout_ticks, a.err, 0, 0};
  w.progress();
  uint64_t done = 0;
  uint32_t rr = 0;
  for (;;) {
    uint64_t r_pos = 0, dst = 0, bytes = 0;
    uint32_t q = 0, k = 0;
    bool stop = done >= u.total_msgs;
    if (wave == 0 && !stop) {
      uint64_t av = 0, ready;
      for (;;) {
        av = mine ? ld_rlx(coord + offsetof(RingCoord, prod)) - hm : 0;
        ready = __ballot(av > 0);
        if (ready) break;
        __builtin_amdgcn_s_sleep(2);
        if (w.expired()) {
          stop = true;
          break;
        }
      }
      order();
      if (!stop) {
        const uint64_t from = ready >> rr;
        q = from ? rr + (uint32_t)__ffsll((unsigned long long)from) - 1
                 : (uint32_t)__ffsll((unsigned long long)ready) - 1;
        const DevRing rg = table(&a.rings[u.first_ring + q]);
        const uint32_t sid = table(&a.stream_of_prod[u.prod_stream_base + q]);
        const DevStream so = table(&a.streams[sid]);
        const uint64_t q_hm = lane64(hm, q), q_out = lane64(out_pos, q), q_cnt = lane64(cnt, q);
        uint64_t n = lane64(av, q);
        if (n > 64) n = 64;
        if (n > rg.E) n = rg.E;
        uint64_t e = 0;
        if (lane < n) {
          uint64_t i = q_hm % rg.E + lane;
          if (i >= rg.E) i -= rg.E;
          e = ld_rlx(rg.entries + 8 * i);
        }
        const uint64_t sz = e & kEntrySizeMask, incl = wave_scan(sz, lane);
        const uint64_t some = __ballot(lane < n && (lane == 0 || incl <= rg.P / 4));
        k = (uint32_t)__popcll(some);  // leading lanes: incl never decreases
        bytes = lane64(incl, k - 1);
        // entries are checked against the plan before any byte moves, so a
        // malformed entry stops the pump instead of writing out of bounds
        const bool bad = lane < k && (sz > rg.P || q_out + incl > so.out_bytes ||
                                      q_cnt + lane >= so.n_msgs);
        if (__ballot(bad)) {
          if (lane == 0)
            raise_error(a.err, kErrCorrupt);
          stop = true;
        } else if (lane < k) {
          if (a.trace) a.trace[so.trace_base + q_cnt + lane] = sid;
          if (a.ts_pop) a.ts_pop[so.first_msg + q_cnt + lane] = wall_clock64();
        }
        r_pos = lane64(pos, q);
        dst = so.out_base + q_out;
      }
    }
    if (WAVES > 1) {
      if (wave == 0 && lane == 0) {
        cast->w[0] = q;
        cast->w[1] = r_pos;
        cast->w[2] = dst;
        cast->w[3] = bytes;
        cast->stop = stop;
      }
      __syncthreads();
      q = (uint32_t)cast->w[0];
      r_pos = cast->w[1];
      dst = cast->w[2];
      bytes = cast->w[3];
      stop = cast->stop;
    }
    if (stop) return;
    Feed<false> f;
    {
      const DevRing rg = table(&a.rings[u.first_ring + q]);
      f.payload = rg.payload;
      f.P = rg.P;
    }
    f.v_size = bytes;
    f.v_pos = r_pos;
    f.v_addr = dst;
    f.j = 1;
    move_feed<WAVES, false>(f, wave, lane);
    if (WAVES > 1) __syncthreads();  // every wave's reads of the ring have returned
    if (wave == 0) {
      if (lane == q) {
        hb += bytes;
        hm += k;
        out_pos += bytes;
        cnt += k;
        pos += bytes;
        if (pos >= f.P) pos -= f.P;
      }
      st_pair(lane64(coord, q) + offsetof(RingCoord, cons), hm, hb, lane == q);
      done += k;
      rr = q + 1 < u.n_rings ? q + 1 : 0;
    }
    w.progress();
  }
}

// A locking MPSC ring consumed by a team of workgroups.  The ring holds one
// total order; it is cut into rounds of consecutive messages.  A member
// claims the next round number; once the previous round is defined the new
// round starts where that one ends and takes up to kLockBatch messages that
// are already published (so a round never waits on room the ring cannot
// give); the member copies it and releases the ring room in round order.
// Each message's ring position and output address come from the record its
// producer wrote before publishing, so a member never needs another round's
// entries (which producers may already be reusing).
constexpr uint32_t kLockBatch = 32;
__device__ void run_lock_team(const PumpArgs &a, uint32_t uid_in, uint32_t wave, uint32_t lane,
                              Cast *cast) {
  const uint32_t uid = __builtin_amdgcn_readfirstlane(uid_in);
  const DevChannel u = table(&a.chans[uid]);
  const DevRing r = table(&a.rings[u.first_ring]);
  const uint64_t tm_a = r.coord + offsetof(RingCoord, prod);
  const uint64_t hm_a = r.coord + offsetof(RingCoord, cons);
  const uint64_t last = r.base_m + u.total_msgs;  // counter after this pump's messages
  uint64_t *rounds = (uint64_t *)u.rounds;
  __builtin_amdgcn_s_setprio(3);
  Watch w{0, a.timeout_ticks, a.err, 0, 0};
  w.progress();
  for (;;) {
    if (wave == 0) {
      bool stop = false;
      uint64_t k = 0;
      if (lane == 0)
        k = __hip_atomic_fetch_add((uint64_t *)u.claim, 1ull, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
      k = shfl64(k, 0);
      uint64_t start = r.base_m;
      if (k > 0) {
        uint64_t v;
        while ((v = uni64(ld_rlx((uint64_t)&rounds[k - 1]))) == 0) {
          __builtin_amdgcn_s_sleep(1);
          if (w.expired()) {
            stop = true;
            break;
          }
        }
        start = v - 1;
      }
      uint64_t end = start;
      if (!stop && start < last) {
        uint64_t tm;
        while ((tm = uni64(ld_rlx(tm_a))) <= start) {
          __builtin_amdgcn_s_sleep(2);
          if (w.expired()) {
            stop = true;
            break;
          }
        }
        if (!stop) {
          order();
          end = start + kLockBatch;
          if (end > tm) end = tm;
          if (end > last) end = last;
          const uint64_t e =
              lane < end - start ? ld_rlx(r.entries + 8 * ((start + lane) % r.E)) : 0;
          const uint64_t incl = wave_scan(e & kEntrySizeMask, lane);
          end = start + __popcll(__ballot(lane < end - start &&
                                          (lane == 0 || incl <= r.P / kLockShare)));
        }
      }
      // round k is defined even when empty: later claimers see where it ends
      if (!stop && lane == 0) st_rlx((uint64_t)&rounds[k], end + 1);
      if (lane == 0) {
        cast->w[0] = start;
        cast->w[1] = end;
        cast->stop = stop || start >= last;
      }
      order();
    }
    __syncthreads();
    if (cast->stop) return;
    const uint64_t start = cast->w[0], n = cast->w[1] - start;
    // every wave reads the round's entries and records (lane i: message i)
    uint64_t sz = 0, pos = 0, out = 0;
    bool bad = false;
    if (lane < n) {
      const uint64_t seq = start + lane;
      const uint64_t e = ld_rlx(r.entries + 8 * (seq % r.E));
      const uint64_t rec = r.side + 24 * (seq - r.base_m);
      const uint64_t mi = ld_rlx(rec + 16);
      sz = e & kEntrySizeMask;
      pos = ld_rlx(rec);
      out = ld_rlx(rec + 8);
      const uint32_t p = (uint32_t)(e >> 48) % u.K;
      const uint32_t sid = a.stream_of_prod[u.prod_stream_base + p];
      const DevStream so = a.streams[sid];
      // checked against the producer's stream before any byte moves
      bad = sz > r.P || out < so.out_base || out - so.out_base > so.out_bytes ||
            sz > so.out_bytes - (out - so.out_base) || mi < so.first_msg ||
            mi - so.first_msg >= so.n_msgs;
      if (wave == 0 && !bad) {
        if (a.trace) a.trace[u.trace_base + (seq - r.base_m)] = sid;
        if (a.ts_pop) a.ts_pop[mi] = wall_clock64();
      }
    }
    if (__ballot(bad)) {
      if (lane == 0)
        raise_error(a.err, kErrCorrupt);
      return;  // the same in every wave
    }
    Feed<false> f;
    f.payload = r.payload;
    f.P = r.P;
    f.v_size = sz;
    f.v_pos = pos % r.P;
    f.v_addr = out;
    f.j = (uint32_t)n;
    move_feed<kPumpBlock / 64, false>(f, wave, lane);
    __syncthreads();  // every wave's reads of the ring have returned
    if (wave == 0) {
      // release in round order
      const uint64_t b_end = n ? lane64(pos, (uint32_t)n - 1) + lane64(sz, (uint32_t)n - 1) : 0;
      bool stop = false;
      while (uni64(ld_rlx(hm_a)) != start) {
        __builtin_amdgcn_s_sleep(1);
        if (w.expired()) {
          stop = true;
          break;
        }
      }
      if (!stop) st_pair(hm_a, start + n, b_end, lane == 0);
      if (lane == 0) cast->late_stop = stop;
    }
    __syncthreads();
    if (cast->late_stop) return;
    w.progress();
  }
}

// A ring with one producer whose two ends are each split over workgroups.
// The stream's messages are cut into groups of consecutive ones: up to
// kSplitMost, and up to P / (teams + 2) of the ring's bytes unless the first is
// larger, so that every team's group fits beside the others' and one to come.  Every member finds the same groups in the size table (the
// consumers check the entries against it).  Group g belongs to team g mod A;
// the B workgroups of a team move a share of its bytes each.  Where a message
// lies in the ring and in the output follows from the sizes before it, so a
// producer member waits for nothing but room, a consumer member for nothing
// but the group's publication; the first member of the team publishes the
// group (or releases its room) once the others have told it of their shares
// and the groups before have been published (released).  No wait is
// circular: the first group that is not published waits for room only, every
// group before it is published, and so its room is released in time.
constexpr uint32_t kSplitMost = 16;

struct Groups {
  const uint64_t *sizes;  // of the stream's messages
  uint64_t n, P, lim;
  uint32_t most;
  uint64_t first = 0;     // message of lane 0
  uint64_t run = 0;       // bytes of the messages before it
  uint64_t size = 0, incl = 0;
  uint32_t lo = 0, hi = 0;  // lanes of the current group
  bool bad = false;         // a size up to the current group's end is impossible
  __device__ __forceinline__ Groups(const PumpArgs &a, const DevStream &st, const DevRing &r,
                                    uint32_t teams, uint32_t lane)
      : sizes(a.msg_size + st.first_msg), n(st.n_msgs), P(r.P), lim(r.P / (teams + 2)),
        most(r.E < kSplitMost ? (uint32_t)r.E : kSplitMost) {
    load(lane);
  }
  __device__ __forceinline__ uint32_t held() const { return n - first < 64 ? n - first : 64; }
  __device__ __forceinline__ void load(uint32_t lane) {
    size = lane < held() ? sizes[first + lane] : 0;
    incl = wave_scan(size, lane);
  }
  // the next group (empty past the last)
  __device__ __forceinline__ void next(uint32_t lane) {
    lo = hi;
    if (lo + most > 64 && first + 64 < n) {
      run += lane64(incl, lo - 1);
      first += lo;
      lo = 0;
      load(lane);
    }
    const bool in = lane >= lo && lane < held() && lane < lo + most &&
                    (lane == lo || incl - before() <= lim);
    hi = lo + (uint32_t)__popcll(__ballot(in));  // leading lanes: incl never decreases
    bad |= __ballot(lane < hi && size > P) != 0;
  }
  // bytes of the messages between lane 0 and the group, and of the group
  __device__ __forceinline__ uint64_t before() const { return lo ? lane64(incl, lo - 1) : 0; }
  __device__ __forceinline__ uint64_t bytes() const { return lane64(incl, hi - 1) - before(); }
  // group number `by` from here
  __device__ __forceinline__ void skip(uint32_t by, uint32_t lane) {
    for (uint32_t i = 0; i < by && (i == 0 || hi > lo); i++) next(lane);
  }
};

// Member t's words beside the ring's base word (DevChannel::claim).
__device__ __forceinline__ uint64_t split_word(uint64_t base_a, uint32_t members, uint32_t end,
                                               uint32_t t) {
  return base_a + 64 + end * ((8 * members + 63) & ~63u) + 8 * t;
}

// The share of a member of a group's bytes: member b's starts at b shares.
// A member without one (the first always takes part) leaves the group alone:
// nobody waits for it, so the group may be published, consumed and its room
// given to later messages before it gets there.
__device__ __forceinline__ uint64_t split_part(uint64_t bytes, uint32_t B) {
  const uint64_t part = (bytes + B - 1) / B;
  return part < kChunkBytes ? kChunkBytes : part;
}
template <bool kToRing>
__device__ __forceinline__ void split_move(const Groups &g, const DevRing &r, uint64_t base_b,
                                           uint64_t addr, uint32_t b, uint32_t B, uint32_t wave,
                                           uint32_t lane) {
  const uint64_t before = g.before(), part = split_part(g.bytes(), B);
  // this lane's message, clipped to the share
  const uint64_t x0 = before + b * part, x1 = x0 + part, m0 = g.incl - g.size;
  const uint64_t c0 = m0 < x0 ? x0 : m0, c1 = g.incl < x1 ? g.incl : x1;
  Feed<kToRing> f;
  f.payload = r.payload;
  f.P = r.P;
  f.v_size = c1 > c0 ? c1 - c0 : 0;
  f.v_pos = (base_b + g.run + c0) % r.P;
  f.v_addr = addr + (c0 - m0);
  f.l = g.lo;
  f.j = g.hi;
  move_feed<kPumpBlock / 64, kToRing>(f, wave, lane);
}

// The first member of a team waits until the others have moved their shares
// of group number `no`.  False when the pump must stop.
__device__ __forceinline__ bool split_gather(uint64_t words, uint64_t bytes, uint32_t B,
                                             uint64_t no, uint32_t lane, Watch &w) {
  const uint64_t part = split_part(bytes, B);
  const bool on = lane > 0 && lane < B && lane * part < bytes;
  w.poll();
  for (;;) {
    const uint64_t left = __ballot(on && ld_rlx(words + 8 * lane) < no + 1);
    if (!left) return true;
    if (w.stuck(left)) return false;
  }
}

__device__ void run_split_producer(const PumpArgs &a, const DevRole &role, uint32_t wave,
                                   uint32_t lane, Cast *cast) {
  const uint32_t A = role.ids[2], B = role.ids[3], t = role.ids[1], team = t / B, b = t - team * B;
  const DevStream st = table(&a.streams[role.ids[0]]);
  const DevRing r = table(&a.rings[st.ring]);
  const uint64_t base_a = table(&a.chans[st.channel].claim);
  const uint64_t words = split_word(base_a, A * B, 0, team * B);
  const uint64_t tm_a = r.coord + offsetof(RingCoord, prod),
                 hm_a = r.coord + offsetof(RingCoord, cons), hb_a = hm_a + 8;
  if (st.n_msgs == 0) return;
  Watch w{0, a.timeout_ticks, a.err, 0, 0};
  w.progress();
  Groups g(a, st, r, A, lane);
  // the ring's byte counter when the pump starts: nothing is published before
  // the first member has read it
  if (wave == 0) {
    uint64_t v = 0;
    bool stop = false;
    if (t == 0) {
      v = uni64(ld_rlx(hb_a)) + 1;
      if (lane == 0) st_rlx(base_a, v);
      if (uni64(ld_rlx(tm_a)) != r.base_m) {  // not what the host planned for
        stop = true;
        if (lane == 0)
          raise_error(a.err, kErrCorrupt);
      }
    } else {
      while ((v = uni64(ld_rlx(base_a))) == 0 && !stop) stop = w.expired();
    }
    if (lane == 0) {
      cast->w[0] = v - 1;
      cast->stop = stop;
    }
  }
  __syncthreads();
  const uint64_t base_b = uni64(cast->w[0]);
  if (cast->stop) return;
  uint64_t no = team;             // group number
  uint64_t pub_m = 0, pub_b = 0;  // the counters that publish the last group
  uint64_t last_bytes = 0;
  uint32_t last_j = 0;            // its messages
  for (g.skip(team + 1, lane);; g.skip(A, lane)) {
    const bool mine = lane >= g.lo && lane < g.hi, more = g.hi > g.lo;
    const uint64_t idx = g.first + lane;
    const uint64_t off = mine ? a.msg_off[st.first_msg + idx] : 0;
    // publish the group before this one: its payload and entries are in
    // place once the stores of every wave of the team have completed
    drain();
    __syncthreads();
    bool stop = false;
    if (wave == 0 && last_j) {
      if (b) {
        if (lane == 0) st_rlx(words + 8 * b, no - A + 1);
      } else {
        stop = !split_gather(words, last_bytes, B, no - A, lane, w);
        w.poll();
        for (uint64_t tm; !stop && (tm = uni64(ld_rlx(tm_a))) != pub_m - last_j;) stop = w.stuck(tm);
        order();
        if (!stop) {
          if (a.ts_push && lane < last_j)
            a.ts_push[st.first_msg + (pub_m - r.base_m) - last_j + lane] = wall_clock64();
          if (lane == 0) {
            st_rlx(tm_a + 8, pub_b);
            st_rlx(tm_a, pub_m);
          }
        }
      }
    }
    w.progress();
    if (!more) return;
    last_bytes = g.bytes();
    last_j = 0;
    no += A;
    if (b && b * split_part(last_bytes, B) >= last_bytes) continue;
    const bool bad = mine && (off > st.src_bytes || g.size > st.src_bytes - off ||
                              g.run + g.incl > st.out_bytes);
    if (g.bad || __ballot(bad)) {  // the same in every wave, before a byte of the group moves
      if (wave == 0 && lane == 0)
        raise_error(a.err, kErrCorrupt);
      return;
    }
    const uint64_t end_m = r.base_m + g.first + g.hi;
    const uint64_t end_b = base_b + g.run + lane64(g.incl, g.hi - 1);
    if (wave == 0) {
      w.poll();
      while (!stop) {
        const uint64_t hm = uni64(ld_rlx(hm_a)), hb = uni64(ld_rlx(hb_a));
        if (end_m - hm <= r.E && end_b - hb <= r.P) break;
        __builtin_amdgcn_s_sleep(1);
        stop = w.stuck(hm + hb);  // (both only grow)
      }
      order();
      if (lane == 0) cast->stop = stop;
    }
    __syncthreads();
    if (cast->stop) return;
    if (b == 0 && wave == 0 && mine)
      st_rlx(r.entries + 8 * ((r.base_m + idx) % r.E), g.size | ((uint64_t)st.producer << 48));
    split_move<true>(g, r, base_b, st.src_base + off, b, B, wave, lane);
    last_j = g.hi - g.lo;
    pub_m = end_m;
    pub_b = end_b;
  }
}

__device__ void run_split_consumer(const PumpArgs &a, const DevRole &role, uint32_t wave,
                                   uint32_t lane, Cast *cast) {
  const uint32_t A = role.ids[2], B = role.ids[3], t = role.ids[1], team = t / B, b = t - team * B;
  const DevChannel u = table(&a.chans[role.ids[0]]);
  const DevRing r = table(&a.rings[u.first_ring]);
  const uint32_t sid = table(&a.stream_of_prod[u.prod_stream_base]);
  const DevStream st = table(&a.streams[sid]);
  const uint64_t words = split_word(u.claim, A * B, 1, team * B);
  const uint64_t tm_a = r.coord + offsetof(RingCoord, prod),
                 hm_a = r.coord + offsetof(RingCoord, cons);
  if (st.n_msgs == 0) return;
  Watch w{0, a.timeout_ticks, a.err, 0, 0};
  w.progress();
  Groups g(a, st, r, A, lane);
  uint64_t no = team;
  for (g.skip(team + 1, lane); g.hi > g.lo; g.skip(A, lane), no += A) {
    const bool mine = lane >= g.lo && lane < g.hi;
    const uint64_t idx = g.first + lane, end_m = r.base_m + g.first + g.hi, bytes = g.bytes();
    if (b && b * split_part(bytes, B) >= bytes) continue;
    if (wave == 0) {
      bool stop = false;
      w.poll();
      for (uint64_t tm; !stop && (int64_t)((tm = uni64(ld_rlx(tm_a))) - end_m) < 0;) {
        __builtin_amdgcn_s_sleep(1);
        stop = w.stuck(tm);
      }
      order();
      if (lane == 0) cast->stop = stop;
    }
    __syncthreads();
    if (cast->stop) return;
    // (the ring's byte counter was there before anything was published)
    const uint64_t base_b = uni64(ld_rlx(u.claim)) - 1;
    const uint64_t e = mine ? ld_rlx(r.entries + 8 * ((r.base_m + idx) % r.E)) : 0;
    // entries are checked against the plan before any byte moves
    const bool bad = mine && ((e & kEntrySizeMask) != g.size || (e >> 48) != st.producer ||
                              g.run + g.incl > st.out_bytes);
    if (g.bad || __ballot(bad)) {  // the same in every wave
      if (lane == 0)
        raise_error(a.err, kErrCorrupt);
      return;
    }
    if (b == 0 && wave == 0 && mine) {
      if (a.trace) a.trace[st.trace_base + idx] = sid;
      if (a.ts_pop) a.ts_pop[st.first_msg + idx] = wall_clock64();
    }
    split_move<false>(g, r, base_b, st.out_base + g.run + g.incl - g.size, b, B, wave, lane);
    __syncthreads();  // every wave's reads of the ring have returned
    if (wave == 0) {
      bool stop = false;
      if (b) {
        if (lane == 0) st_rlx(words + 8 * b, no + 1);
      } else {
        const uint64_t start = end_m - (g.hi - g.lo);
        stop = !split_gather(words, bytes, B, no, lane, w);
        w.poll();
        for (uint64_t hm; !stop && (hm = uni64(ld_rlx(hm_a))) != start;) stop = w.stuck(hm);
        order();
        if (!stop)
          st_pair(hm_a, end_m, base_b + g.run + lane64(g.incl, g.hi - 1), lane == 0);
      }
      if (lane == 0) cast->late_stop = stop;
    }
    __syncthreads();
    if (cast->late_stop) return;
    w.progress();
  }
}

// kSplit: the rings that have one producer are split (no endpoint is a wave
// or a workgroup of its own but a locking ring's).  The forms are two kernels to
// keep the split ends' spills (7 VGPRs, 24 B of scratch, 182 SGPRs to lanes) out
// of the other one, which spills 113 SGPRs to lanes and has no scratch; one
// kernel with all of them needs 28 B and 200.
template <bool kSplit>
__global__ __launch_bounds__(kPumpBlock) __attribute__((amdgpu_waves_per_eu(6, 8)))
void pump_kernel(PumpArgs a) {
  __shared__ Cast cast;
  const DevRole role = table(&a.roles[blockIdx.x]);
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform in the wave
  if (role.kind == kRoleLockMember) {
    run_lock_team(a, role.ids[0], wave, lane, &cast);
  } else if (role.kind == kRoleProducerGroup) {
    run_producer<kPumpBlock / 64>(a, role.ids[0], wave, lane, &cast);
  } else if constexpr (kSplit) {
    if (role.kind == kRoleProducerSplit)
      run_split_producer(a, role, wave, lane, &cast);
    else
      run_split_consumer(a, role, wave, lane, &cast);
  } else if (role.kind == kRoleProducerWaves) {
    if (wave < role.count) run_producer<1>(a, a.roles[blockIdx.x].ids[wave], 0, lane, nullptr);
  } else if (role.kind == kRoleConsumerWaves) {
    if (wave < role.count) run_consumer<1>(a, a.roles[blockIdx.x].ids[wave], 0, lane, nullptr);
  } else {
    run_consumer<kPumpBlock / 64>(a, role.ids[0], wave, lane, &cast);
  }
}

// Host-API push: copy the payload into the ring, write the entries, then
// publish the new message counter into host-coherent memory.  Written through
// like a pump's payload and waited for instead of a system-scope fence; a
// workgroup takes kPushPart bytes, since one copies only 25 GB/s, and the
// last of them publishes (the pushes of a context run one after another, so
// they share one arrival counter).  32 messages of 512 KiB pushed and taken
// out: 660 us with one workgroup and the fence, 337 now; messages of a few
// KiB are bound by their launches (5.5 us a message either way).
constexpr uint32_t kPushPart = 16384, kPushGroups = 64;
__global__ __launch_bounds__(256) void push_kernel(PushArgs a) {
  const uint32_t tid = threadIdx.x;
  const uint64_t lo = a.bytes * blockIdx.x / gridDim.x, hi = a.bytes * (blockIdx.x + 1) / gridDim.x;
  Feed<true> f;
  f.payload = a.ring.payload;
  f.P = a.ring.P;
  f.v_size = hi - lo;
  f.v_pos = (a.pos + lo) % a.ring.P;
  f.v_addr = a.src + lo;
  f.j = 1;
  move_feed<4, true>(f, __builtin_amdgcn_readfirstlane(tid >> 6), tid & 63);
  for (uint32_t i = blockIdx.x * 256 + tid; i < a.n_entries; i += gridDim.x * 256)
    st_rlx(a.ring.entries + 8 * ((a.first_entry + i) % a.ring.E),
           a.entry_bytes | ((uint64_t)a.producer << 48));
  drain();
  __syncthreads();
  if (tid) return;
  if (gridDim.x > 1) {
    if (__hip_atomic_fetch_add(a.arrive, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) !=
        gridDim.x - 1)
      return;
    __hip_atomic_store(a.arrive, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    drain();
  }
  __hip_atomic_store(a.publish, a.publish_value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

hipError_t launch_pump(const PumpArgs &a, bool split, uint32_t n_wgs, hipStream_t stream) {
  hipLaunchKernelGGL(split ? pump_kernel<true> : pump_kernel<false>, dim3(n_wgs),
                     dim3(kPumpBlock), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_push(const PushArgs &a, hipStream_t stream) {
  const uint64_t parts = (a.bytes + kPushPart - 1) / kPushPart;
  const uint32_t grid = parts < 1 ? 1 : parts > kPushGroups ? kPushGroups : (uint32_t)parts;
  hipLaunchKernelGGL(push_kernel, dim3(grid), dim3(256), 0, stream, a);
  return hipGetLastError();
}

// (both forms may be in flight together)
int pump_occupancy(int *wgs_per_cu) {
  int split = 0;
  int e = (int)hipOccupancyMaxActiveBlocksPerMultiprocessor(wgs_per_cu, pump_kernel<false>,
                                                            kPumpBlock, 0);
  if (e == 0)
    e = (int)hipOccupancyMaxActiveBlocksPerMultiprocessor(&split, pump_kernel<true>, kPumpBlock, 0);
  if (split < *wgs_per_cu) *wgs_per_cu = split;
  return e;
}

}  // namespace hicr
