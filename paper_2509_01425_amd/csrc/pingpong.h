// pingpong.h -- arguments of the two-endpoint ping-pong kernel.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hicr {

// Counter words of one launch with W workgroups per endpoint, zeroed before
// it, one 128-byte line each: the four channel counters, then (W >
// kPingPongDirect) four counters per group of kPingPongDirect workgroups, and
// a line of flags per workgroup.
constexpr uint32_t kPingPongDirect = 16;
constexpr size_t kLineWords = 16;
__host__ __device__ inline size_t pingpong_groups(uint32_t W) { return (W + kPingPongDirect - 1) / kPingPongDirect; }
inline size_t pingpong_words(uint32_t W) {
  return kLineWords * (4 + (W > kPingPongDirect ? 4 * pingpong_groups(W) + 2 * (size_t)W : 0));
}

struct PingPongArgs {
  uint64_t src, dst, ring_a, ring_b, buf;  // 16-byte aligned device addresses
  uint64_t size;                            // message bytes
  uint32_t W;                               // workgroups per endpoint
  uint32_t reps;                            // round trips
  uint64_t *ctr;      // [pingpong_words(W)], 128-byte aligned; channel counters:
                      // A arrived, A freed, B arrived, B freed (stripes)
  uint64_t *t_start;  // [reps] pinger clock before each push (100 MHz)
  uint64_t *t_end;    // [reps] pinger clock after reading each echo
  uint32_t *err;      // time-out flag
  uint64_t timeout_ticks;
};

hipError_t launch_pingpong(const PingPongArgs &a, hipStream_t s);
int pingpong_occupancy(int *wgs_per_cu);

}  // namespace hicr
