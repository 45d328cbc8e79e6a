// internal.h -- structures shared by the host runtime and the gfx950 kernels
// of the copy engine.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "stream_plan.h"

namespace hicr {

constexpr int kCopyBlock = 256;         // threads per copy workgroup (4 waves)
constexpr int kScanBlock = 1024;        // threads of the one scan workgroup
constexpr uint32_t kMaxLdsDescs = 4096; // requests scanned into LDS by every copy workgroup
static_assert(kMaxLdsDescs == kStreamMaxReqs, "a batch of more requests has its table in memory");
constexpr uint32_t kTile = 4096;        // requests per tile of a scanned table
constexpr uint32_t kMaxTiles = 4096;    // tiles per launch over a scanned table
constexpr uint32_t kLineBytes = 128;    // interior piece boundaries are line aligned
constexpr uint32_t kMinSplit = 1024;    // never split a request below 1 KiB pieces

// Device-side batch: structure of arrays, uploaded in one copy.  Addresses
// are already resolved from (slot, offset) on the host.
struct DevBatch {
  const uint64_t *dst;   // [n] destination byte address
  const uint64_t *src;   // [n] source byte address
  const uint64_t *size;  // [n] bytes
  const uint64_t *slots; // [n] dst_slot | (uint64_t)src_slot << 32
  uint32_t n;
};

// How a copy launch tells the host that it has ended.  Every workgroup waits
// for its own stores, which write through to the device's coherence point;
// then a launch of at most kDoneWords workgroups stores seq to one word of
// pinned host memory per workgroup, and a larger one counts its workgroups in
// *arrive (device memory, zero before and after every launch), the last of
// them storing to words[0].  words null: no signal.
constexpr uint32_t kDoneWords = 64;
struct Done {
  uint64_t *words = nullptr;
  uint32_t *arrive = nullptr;
  uint64_t seq = 0;
};
inline uint32_t done_words(uint32_t grid) { return grid <= kDoneWords ? grid : 1; }

// Schedule as the kernel sees it.
struct DevSched {
  uint32_t chunk, wgs, unroll, cls;
};

// ceil(a / b), in 32-bit arithmetic when both fit (a 64-bit division is
// several times longer on the GPU).
__host__ __device__ inline uint64_t div_up(uint64_t a, uint64_t b) {
  if (a == 0) return 0;
  if (((a | b) >> 32) == 0) return 1 + ((uint32_t)a - 1) / (uint32_t)b;
  return 1 + (a - 1) / b;
}

// Piece length for one request under (chunk, wgs): pieces start at line
// boundaries of the destination (except the first), so a piece never shares
// a 16-byte store with its neighbour inside one request.
__host__ __device__ inline uint64_t piece_len(uint64_t dst, uint64_t size, uint32_t chunk,
                                              uint32_t wgs) {
  uint64_t span = dst + size - (dst & ~(uint64_t)(kLineBytes - 1));
  uint64_t L = chunk;
  if (wgs > 1 && span < (uint64_t)wgs * chunk) {
    uint64_t per = div_up(span, wgs);
    per = (per + kLineBytes - 1) & ~(uint64_t)(kLineBytes - 1);
    if (per < kMinSplit) per = kMinSplit;
    if (per < L) L = per;
  }
  return L;
}

__host__ __device__ inline uint64_t piece_count(uint64_t dst, uint64_t size, uint32_t chunk,
                                                uint32_t wgs) {
  if (size == 0) return 1;  // a zero-byte request still completes (and counts) once
  uint64_t span = dst + size - (dst & ~(uint64_t)(kLineBytes - 1));
  return div_up(span, piece_len(dst, size, chunk, wgs));
}

// Launch the fused copy kernel over one sub-batch (n <= kMaxLdsDescs), piece
// table scanned in LDS by every workgroup.
hipError_t launch_copy(const DevBatch &b, DevSched s, uint32_t grid, hipStream_t stream);
// Raise the words of `done` (armed for one workgroup) once everything before it has ended.
hipError_t launch_done(Done done, hipStream_t stream);
// Scan the pieces of a batch (1 <= n <= kTile * kMaxTiles, fewer than 2^31
// pieces) into a tiled table: ends[0, n) holds each tile's inclusive prefix
// relative to the tile, tile_tot[0, ceil(n / kTile)) the tile totals.  staged:
// the requests lie there in pinned host memory, and are moved to b first.
hipError_t launch_scan(const DevBatch *staged, const DevBatch &b, DevSched s, uint32_t *ends,
                       uint32_t *tile_tot, hipStream_t stream);
// Move bytes (a multiple of 8) of pinned host memory to device memory.
hipError_t launch_upload(const void *h_dev, void *d, uint64_t bytes, hipStream_t stream);
// Launch the copy kernel over a batch whose table launch_scan has written.
hipError_t launch_copy_mem(const DevBatch &b, DevSched s, const uint32_t *ends,
                           const uint32_t *tile_tot, uint32_t grid, Done done,
                           hipStream_t stream);
// Copy requests [0, n) as one stream shared evenly by `waves` wavefronts: wave w moves what lies between starts[w] and starts[w + 1]
// (starts[waves] = {0, n}).  dst, src, size and starts may lie in pinned host
// memory.
inline uint32_t stream_grid(uint32_t waves) { return (waves + kCopyBlock / 64 - 1) / (kCopyBlock / 64); }
hipError_t launch_stream(const DevBatch &b, const StreamStart *starts, uint32_t waves, Done done,
                         hipStream_t stream);
// The same for up to kArgReqs requests, which go into the kernel's arguments.
// h holds n destinations, sources and sizes, which count for `load` in all
// (stream_load); args_fit says whether they can go that way, and the lowest of
// both addresses.
constexpr uint32_t kArgReqs = 256;
bool args_fit(const uint64_t *h, uint64_t n, uint64_t load, uint64_t *dst, uint64_t *src);
hipError_t launch_stream_args(const uint64_t *h, uint32_t n, uint64_t dst, uint64_t src,
                              uint64_t load, uint32_t waves, Done done, hipStream_t stream);
// Raise the slot counters of n requests (slots[i] = dst | src << 32); queued
// after the copy launches of the same requests on the same stream.
inline uint32_t count_grid(uint64_t n) { return (uint32_t)((n + 1023) / 1024); }
hipError_t launch_count(const uint64_t *slots, uint64_t n, uint64_t *counters, Done done,
                        hipStream_t stream);
// Workgroups of the copy kernel that one CU holds at once.
int copy_occupancy(int *wgs_per_cu);

}  // namespace hicr
