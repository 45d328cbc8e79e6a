// pingpong.hip -- the ping-pong benchmark of the paper's Test Case 1 on one
// GPU: two endpoints connected by two opposing channels of one-message
// capacity.  The pinger pushes a message into channel A and waits for its
// echo on channel B; the ponger takes each message from A into its own
// buffer, frees A, and pushes the buffer into B once the pinger has freed B.
//
// Each endpoint is a group of W workgroups: message bytes are striped over
// the group (workgroup w owns stripe w), and each channel's counters count
// stripes -- a channel's tail (`arrived`) and head (`freed`) advance by W per
// message, so a message is visible once all of its stripes are, and a ring
// is free once every stripe has been read.  W = 1 is a single workgroup per
// endpoint; large messages use many so the copies run at memory speed.
//
// What the endpoints exchange moves with agent-scope accesses (sc1: see
// channel.hip), so a workgroup counts a stripe once its own stores have
// completed and no fence is needed on either side.  Bound by the two copies
// of each one-way, one behind the other, and by ~2 us of counter round trips.
// One-way, with fences and one counter that all workgroups poll -> now: 1 B
// 2.4 -> 2.0 us, 64 KiB 8.3 -> 3.0, 1 MiB 9.5 -> 4.9, 16 MiB 60.6 -> 10.2,
// 64 MiB 99 -> 32.5 (256 MiB of copies: 8.3 TB/s, the rings held by the
// memory-side cache).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pingpong.h"
#include "span.h"

namespace hicr {

// Copy bytes [lo, hi) of a message with a workgroup of four waves, chunk by
// chunk in turn (chunk boundaries on destination lines, so the first chunk is
// shorter when lo is off them).
template <int LP, int SP>
__device__ __forceinline__ void stripe_copy(uint64_t d, uint64_t s, uint64_t lo, uint64_t hi,
                                            uint32_t wave, uint32_t lane) {
  const uint64_t base = lo - ((d + lo) & (kLineBytes - 1));  // (may wrap below zero)
  uint64_t c = wave;
  move_chunks<LP, SP>(
      [&]() {
        const uint64_t at = c ? base + c * kChunkBytes : lo;
        const uint64_t end = base + (c + 1) * kChunkBytes < hi ? base + (c + 1) * kChunkBytes : hi;
        c += 4;
        return Chunk{d + at, s + at, at < end ? (uint32_t)(end - at) : 0u};
      },
      lane);
}

__device__ __forceinline__ bool wait_at_least(const uint64_t *ctr, uint64_t v, uint64_t deadline,
                                              uint32_t *err) {
  while (__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < v) {
    __builtin_amdgcn_s_sleep(1);
    if (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return false;
    if (wall_clock64() > deadline) {
      __hip_atomic_fetch_or(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return false;
    }
  }
  return true;
}

__global__ __launch_bounds__(256) void pingpong_kernel(PingPongArgs a) {
  __shared__ uint32_t ok, last;
  const uint32_t t = threadIdx.x, lane = t & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const bool pinger = blockIdx.x < a.W;
  const uint32_t w = pinger ? blockIdx.x : blockIdx.x - a.W;
  // stripe w of an s-byte message: whole lines, the last takes the rest
  const uint64_t stripe =
      ((a.size + a.W - 1) / a.W + kLineBytes - 1) & ~(uint64_t)(kLineBytes - 1);
  const uint64_t lo = (uint64_t)w * stripe < a.size ? (uint64_t)w * stripe : a.size;
  const uint64_t hi = lo + stripe < a.size ? lo + stripe : a.size;
  const uint64_t W = a.W;
  uint64_t deadline = wall_clock64() + a.timeout_ticks;
  // an earlier launch of the same call has timed out: so does this one
  if (t == 0) ok = !__hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (!ok) return;
  __syncthreads();
  // Channel counter c (0 A arrived, 1 A freed, 2 B arrived, 3 B freed): all
  // stripes of message m have been counted.  With few workgroups everybody
  // polls the counter itself.  With more, hundreds of pollers of one line hold
  // up the very atomics they wait for, which also queue on it one by one; so
  // the count goes through a counter per kPingPongDirect workgroups, and who
  // completes it writes m + 1 to every waiting workgroup's own line.
  const bool direct = a.W <= kPingPongDirect;
  uint64_t *const groups = a.ctr + 4 * kLineWords;
  uint64_t *const flags = groups + 4 * kLineWords * pingpong_groups(a.W);
  // thread 0 polls, and the barrier orders every other wave's later accesses
  // after that
  auto wait = [&](uint32_t c, uint64_t messages) {
    if (t == 0) {
      const uint64_t *p = direct ? a.ctr + kLineWords * c : flags + kLineWords * blockIdx.x + c;
      ok = wait_at_least(p, direct ? messages * W : messages, deadline, a.err);
    }
    __syncthreads();
    return ok != 0;
  };
  // every wave's copies have completed before one stripe is counted
  auto add = [](uint64_t *p) {
    return __hip_atomic_fetch_add(p, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
  };
  auto signal = [&](uint32_t c, uint64_t message) {
    drain();
    __syncthreads();
    if (direct) {
      if (t == 0) (void)add(a.ctr + kLineWords * c);
      return;
    }
    if (t == 0) {
      const uint32_t g = w / kPingPongDirect;
      const uint64_t in_group = min(a.W - g * kPingPongDirect, kPingPongDirect);
      const uint64_t n = message + 1;
      last = add(groups + kLineWords * (4 * g + c)) == n * in_group &&
             add(a.ctr + kLineWords * c) == n * pingpong_groups(a.W);
    }
    __syncthreads();
    if (!last) return;
    // the pinger waits for A freed and B arrived, the ponger for the others
    const uint32_t base = c == 1 || c == 2 ? 0 : a.W;
    for (uint32_t i = t; i < a.W; i += 256)
      __hip_atomic_store(flags + kLineWords * (base + i) + c, message + 1, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
  };
  // into a ring, out of a ring
  auto put = [&](uint64_t ring, uint64_t from) {
    stripe_copy<0, kAgent>(ring, from, lo, hi, wave, lane);
  };
  auto get = [&](uint64_t to, uint64_t ring) {
    stripe_copy<kAgentStream, 0>(to, ring, lo, hi, wave, lane);
  };
  for (uint32_t k = 0; k < a.reps; k++) {
    if (pinger) {
      if (w == 0 && t == 0) a.t_start[k] = wall_clock64();
      if (!wait(1, k)) return;      // A is free of message k-1
      put(a.ring_a, a.src);
      signal(0, k);                 // A: stripe arrived
      if (!wait(2, k + 1)) return;  // B holds the echo
      get(a.dst, a.ring_b);
      signal(3, k);                 // B: stripe freed
      if (w == 0 && t == 0) a.t_end[k] = wall_clock64();
    } else {
      if (!wait(0, k + 1)) return;  // A holds message k
      get(a.buf, a.ring_a);
      signal(1, k);                 // A: stripe freed
      if (!wait(3, k)) return;      // B is free of message k-1
      put(a.ring_b, a.buf);
      signal(2, k);                 // B: stripe arrived
    }
    deadline = wall_clock64() + a.timeout_ticks;
  }
}

hipError_t launch_pingpong(const PingPongArgs &a, hipStream_t s) {
  hipLaunchKernelGGL(pingpong_kernel, dim3(2 * a.W), dim3(256), 0, s, a);
  return hipGetLastError();
}

int pingpong_occupancy(int *wgs_per_cu) {
  return (int)hipOccupancyMaxActiveBlocksPerMultiprocessor(wgs_per_cu, pingpong_kernel, 256, 0);
}

}  // namespace hicr
