// span.h -- buffer accesses to one contiguous span of memory (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace hicr {

// Global address space (1): plain global_load/global_store instead of flat.
#define GLOBAL __attribute__((address_space(1)))

typedef int32_t v4i __attribute__((ext_vector_type(4)));
typedef __amdgpu_buffer_rsrc_t rsrc_t;

// A buffer resource over [base, base + bytes): accesses at or past `bytes`
// read zero and write nothing (the hardware's range check), which lets a
// copy loop run whole rounds without clamping its last one.  base and bytes
// are the same in every lane; base may have any alignment (gfx950 runs the
// HSA unaligned-access mode).
__device__ __forceinline__ rsrc_t span_rsrc(uint64_t base, uint32_t bytes) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)base);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32));
  return __builtin_amdgcn_make_buffer_rsrc((void *)(((uint64_t)hi << 32) | lo), (short)0,
                                           (int)__builtin_amdgcn_readfirstlane(bytes),
                                           0x00020000);
}

// Accesses with a cache policy (gfx950 bits: 1 = sc0, 2 = nt, 16 = sc1).
template <int Policy>
__device__ __forceinline__ v4i bload(rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, Policy);
}
template <int Policy>
__device__ __forceinline__ void bstore(rsrc_t r, uint32_t off, v4i v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, Policy);
}
template <int Policy>
__device__ __forceinline__ uint32_t bload8(rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b8(r, off, 0, Policy);
}
template <int Policy>
__device__ __forceinline__ void bstore8(rsrc_t r, uint32_t off, uint32_t v) {
  __builtin_amdgcn_raw_buffer_store_b8((unsigned char)v, r, off, 0, Policy);
}

// Cache policies: read once (nt); agent scope (sc1: visible device-wide once
// the wave has waited for it, and never a stale line); the same, streaming.
constexpr int kReadStream = 2;
constexpr int kAgent = 16;
constexpr int kAgentStream = 18;

// A value that is the same in every lane, in scalar registers.
__device__ __forceinline__ uint64_t uni64(uint64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return ((uint64_t)hi << 32) | lo;
}

// Lane `lane` (uniform) of a 64-bit value held in every lane's registers.
__device__ __forceinline__ uint64_t lane64(uint64_t v, uint32_t lane) {
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), lane);
  return ((uint64_t)hi << 32) | lo;
}

// Nothing the compiler sees moves across this point.
__device__ __forceinline__ void order() { asm volatile("" ::: "memory"); }

// Wait until this wave's memory accesses have completed: its agent-scope
// stores are then visible to every other wave of the device.
__device__ __forceinline__ void drain() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Tell the host that this workgroup's copies have ended (see Done).  Every
// thread of the workgroup calls it, after its last store.
__device__ __forceinline__ void signal_done(const Done &d) {
  if (!d.words) return;
  drain();
  __syncthreads();
  if (threadIdx.x) return;
  if (gridDim.x > kDoneWords) {
    const uint32_t before =
        __hip_atomic_fetch_add(d.arrive, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (before != gridDim.x - 1) return;
    __hip_atomic_store(d.arrive, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    drain();
  }
  uint64_t *w = d.words + (gridDim.x > kDoneWords ? 0 : blockIdx.x);
  __hip_atomic_store(w, d.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// n bytes d <- s (uniform), at most kChunkBytes of destination lines.
constexpr int kChunkRows = 4;  // 1 KiB rows
constexpr uint32_t kChunkBytes = 1024u * kChunkRows;
struct Chunk {
  uint64_t d, s;
  uint32_t n;
};

// A chunk on its way: the 16-byte destination vectors of its rows (a row is
// eight whole lines of the destination: write-through stores of rows across
// lines would write each line twice), and in
// lanes 0-15 the at most 15 bytes before the first, in lanes 16-31 the at
// most 15 bytes after the last of them.  Loads and stores of what a chunk
// does not have are out of the buffer resource's range: they read zero and
// write nothing.  So a chunk costs the same instructions whatever its length
// (also 0), and the compiler can count exactly which of them a store waits
// for; with a branch around the loads it waits for all of them.
template <int LP, int SP>
struct Flight {
  v4i v[kChunkRows];
  uint32_t byte;
  __device__ __forceinline__ static uint32_t head(const Chunk &c) {
    const uint32_t h = (uint32_t)(-c.d) & 15u;
    return h < c.n ? h : c.n;
  }
  // (lanes past the tail get offsets past the chunk by themselves)
  __device__ __forceinline__ static uint32_t byte_off(const Chunk &c, uint32_t lane) {
    const uint32_t nh = head(c), body = nh + ((c.n - nh) & ~15u);
    const uint32_t h = lane < nh ? lane : ~0u;
    return lane < 16 ? h : body + lane - 16;
  }
  // (lanes before the first vector get offsets below zero, past the chunk too)
  __device__ __forceinline__ static uint32_t row_off(const Chunk &c, uint32_t nh, uint32_t lane) {
    return nh + 16 * lane - (((uint32_t)c.d + nh) & (kLineBytes - 1));
  }
  __device__ __forceinline__ void load(const Chunk &c, uint32_t lane) {
    const uint32_t nh = head(c), body = nh + ((c.n - nh) & ~15u), o = row_off(c, nh, lane);
    const rsrc_t r = span_rsrc(c.s, body);
    byte = bload8<LP>(span_rsrc(c.s, c.n), byte_off(c, lane));
#pragma unroll
    for (int k = 0; k < kChunkRows; k++) v[k] = bload<LP>(r, o + 1024u * k);
  }
  __device__ __forceinline__ void store(const Chunk &c, uint32_t lane) const {
    const uint32_t nh = head(c), body = nh + ((c.n - nh) & ~15u), o = row_off(c, nh, lane);
    const rsrc_t r = span_rsrc(c.d, body);
#pragma unroll
    for (int k = 0; k < kChunkRows; k++) bstore<SP>(r, o + 1024u * k, v[k]);
    bstore8<SP>(span_rsrc(c.d, c.n), byte_off(c, lane), byte);
  }
};

// Copy the chunks that next() gives (n = 0 once there are no more) with one
// wave, the next chunk's loads issued before the current chunk's stores.  On
// return every load has completed; stores may still be in flight.
template <int LP, int SP, class Next>
__device__ __forceinline__ void move_chunks(Next next, uint32_t lane) {
  Chunk a = next();
  if (a.n == 0) return;
  Flight<LP, SP> fa, fb;
  fa.load(a, lane);
  do {
    const Chunk b = next();
    fb.load(b, lane);
    fa.store(a, lane);
    a = next();
    fa.load(a, lane);
    fb.store(b, lane);
  } while (a.n);
  order();
}

}  // namespace hicr
