// copy.hip -- fused batched memcpy for gfx950 (CDNA4).
//
// One launch moves a batch of memcpy(dst, dstOff, src, srcOff, size) requests
// (HiCR Sec. 3.1.4) with a persistent grid.  There are three, by the batch:
//   stream_kernel    up to 4,096 requests and about 256 MiB: the host has cut
//                    the batch into equal shares of bytes, one per wave;
//   copy_kernel      up to 4,096 requests, larger: a global index space of
//                    pieces, the inclusive prefix of the pieces per request
//                    scanned by every workgroup into LDS (wavefront scans with
//                    __shfl_up, then a cross-wave carry); wave w of workgroup
//                    g takes pieces 4g + w, 4g + w + 4G, ... and finds each
//                    piece's request by a 64-ary ballot search;
//   copy_kernel_mem  more requests: the prefix is scanned once, by
//                    scan_kernel, one workgroup per tile of 4,096 requests;
//                    every wave takes one contiguous range of pieces, finds
//                    where it starts and ends by the same search, and copies
//                    it as a stream.
// A piece of copy_kernel is copied with buffer loads (at whatever alignment
// the source has: gfx950 runs the HSA unaligned-access mode) and 16-byte
// destination-aligned buffer stores, both non-temporal, in rounds of
// 4 x `unroll` 1 KiB rows, the next round's loads issued before the current
// round's stores (see copy_span); a stream in chunks of 4 KiB of destination
// lines (see Flight).  The at most 15 bytes before the first and after the
// last aligned destination vector are copied byte by byte, so no store ever
// touches a byte outside the request.
//
// The stores of streams write through to the device's coherence point (agent
// scope), so a workgroup that has waited for its stores has nothing to write
// back and can say that it has ended (signal_done): no counter kernel and no
// event behind the copy.  (An agent-scope release in every workgroup, which stores
// that stay in the L2 need, writes back the whole L2 of the XCD and cost more
// than the copy itself on batches of small requests.)
#include <algorithm>

#include "internal.h"
#include "span.h"

namespace hicr {

// Cache policy of the body's buffer accesses (gfx950 bits: 1 = sc0, 2 = nt,
// 16 = sc1).  Neither side is touched again by the copy, so the source is
// read non-temporally and the destination written non-temporally at device
// scope.
constexpr int kLoadPolicy = 2;
constexpr int kStorePolicy = 18;
// Streamed ranges read with the plain policy: the rows of small or unaligned
// requests share source lines with their neighbours, which the caches then
// serve (halo exchange 145 us against 151 us read non-temporally; 8,192
// requests of 256 B - 64 KiB 94-99 against 110 us a pass).
constexpr int kPlainLoad = 0;
// Pieces of at most this many vector bytes take body_small.
constexpr uint32_t kSmallPiece = 8192;

// nb bytes (a multiple of 16) from rs to rd in rounds of U vector rows (1 KiB
// per row), two rounds in flight: round k + 1 is loaded before round k is
// stored, so a wave never waits for a round's loads with nothing else
// outstanding.  Offsets past nb read zero and store nothing.
template <int U>
__device__ __forceinline__ void body(rsrc_t rs, rsrc_t rd, uint32_t nb, uint32_t lane) {
  constexpr uint32_t R = 1024u * U;
  const uint32_t l16 = 16u * lane;
  v4i a[U], c[U];
#pragma unroll
  for (int k = 0; k < U; k++) a[k] = bload<kLoadPolicy>(rs, l16 + 1024u * k);
  for (uint32_t b = 0; b < nb; b += 2 * R) {
#pragma unroll
    for (int k = 0; k < U; k++) c[k] = bload<kLoadPolicy>(rs, b + R + l16 + 1024u * k);
#pragma unroll
    for (int k = 0; k < U; k++) bstore<kStorePolicy>(rd, b + l16 + 1024u * k, a[k]);
#pragma unroll
    for (int k = 0; k < U; k++) a[k] = bload<kLoadPolicy>(rs, b + 2 * R + l16 + 1024u * k);
#pragma unroll
    for (int k = 0; k < U; k++) bstore<kStorePolicy>(rd, b + R + l16 + 1024u * k, c[k]);
  }
}

// Small pieces (the ends of large requests) with plain global accesses: rounds
// of 4 vector rows, indices past the last vector clamped to it (a repeated vector
// rewrites equal bytes).
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef v4u v4u_any __attribute__((aligned(1)));  // 16 bytes at any alignment
__device__ __forceinline__ void body_small(uint64_t d, uint64_t s, uint32_t nv, uint32_t lane) {
  for (uint32_t b = 0; b < nv; b += 256) {
    uint64_t o[4];
#pragma unroll
    for (int k = 0; k < 4; k++) {
      const uint32_t i = b + lane + 64u * k;
      o[k] = 16ull * (i < nv ? i : nv - 1);
    }
    v4u r[4];
#pragma unroll
    for (int k = 0; k < 4; k++) r[k] = *(const GLOBAL v4u_any *)(s + o[k]);
#pragma unroll
    for (int k = 0; k < 4; k++) __builtin_nontemporal_store(r[k], (GLOBAL v4u *)(d + o[k]));
  }
}

// Copy destination bytes [lo, hi) from source address s (the source byte of
// lo) with one wavefront: the 16-byte destination vectors [a0, a1) by body<U>
// (loads at the source's own alignment; body_small for at most 8 KiB of
// vectors), and the at most 15 head bytes
// [lo, a0) and 15 tail bytes [a1, hi) one by one.  Every lane copies one byte
// (lanes 0-15 the head bytes, 16-31 the tail bytes, repeating the last one of
// a range, or byte lo when a range is empty; the other lanes byte lo), so
// repeated stores write equal values inside the piece; the byte is loaded
// before the vectors and stored after them, so its latency overlaps theirs.
// A piece is at most 1 GiB (the chunk limit), so offsets inside it fit 32
// bits.
template <int U>
__device__ __forceinline__ void copy_span(uint64_t lo, uint64_t hi, uint64_t s, uint32_t lane) {
  uint64_t a0 = (lo + 15) & ~(uint64_t)15;
  if (a0 > hi) a0 = hi;
  uint64_t a1 = hi & ~(uint64_t)15;
  if (a1 < a0) a1 = a0;
  const uint64_t nh = a0 - lo, nt = hi - a1;
  uint64_t bo = 0;  // this lane's byte, as an offset from lo
  if (lane < 16)
    bo = nh ? (lane < nh ? lane : nh - 1) : 0;
  else if (lane < 32)
    bo = nt ? (a1 - lo) + (lane - 16 < nt ? lane - 16 : nt - 1) : 0;
  // (lo and hi are the same in every lane: a piece without head or tail
  // bytes, such as an aligned row, skips the byte copy altogether)
  const bool bytes = (nh | nt) != 0;
  unsigned char byte = 0;
  if (bytes) byte = *(const GLOBAL unsigned char *)(s + bo);
  const uint32_t nb = (uint32_t)(a1 - a0);
  if (nb > kSmallPiece)
    body<U>(span_rsrc(s + nh, nb), span_rsrc(a0, nb), nb, lane);
  else if (nb)
    body_small(a0, s + nh, nb >> 4, lane);
  if (bytes) *(GLOBAL unsigned char *)(lo + bo) = byte;
}

__device__ __forceinline__ void copy_range(uint64_t lo, uint64_t hi, uint64_t s, uint32_t unroll,
                                           uint32_t lane) {
  // rounds of 4 x unroll rows (1 KiB each), two rounds in flight: 32 KiB
  // per wave at unroll 4 (on the batched workload 1.5-2 % faster than
  // 16 KiB; byte-misaligned sources of many MiB run better at unroll 2)
  if (unroll >= 4)
    copy_span<16>(lo, hi, s, lane);
  else
    copy_span<8>(lo, hi, s, lane);
}

// First index i in [0, n) with ends[i] > q (ends strictly increasing, q <
// ends[n-1]; ends in LDS or device memory).  Every lane of the wave returns
// the same value.
template <typename Ends>
__device__ __forceinline__ uint32_t find_piece_owner(Ends ends, uint32_t n, uint32_t q,
                                                     uint32_t lane) {
  uint32_t lo = 0, hi = n;
  while (hi - lo > 64) {
    uint32_t step = (hi - lo + 63) >> 6;
    uint32_t idx = lo + (lane + 1) * step - 1;
    bool gt = (idx >= hi - 1) ? true : (ends[idx] > q);
    uint64_t m = __ballot(gt);
    uint32_t f = (uint32_t)__ffsll((unsigned long long)m) - 1;
    uint32_t nlo = lo + f * step;
    uint32_t nhi = lo + (f + 1) * step;
    hi = nhi < hi ? nhi : hi;
    lo = nlo;
  }
  uint32_t idx = lo + lane;
  bool gt = (idx >= hi - 1) ? true : (ends[idx] > q);
  uint64_t m = __ballot(gt);
  return lo + (uint32_t)__ffsll((unsigned long long)m) - 1;
}

// Piece j (of length L) of the request dst <- src, size bytes: pieces start
// at line boundaries of the destination, the first and last clipped to the
// request.
__device__ __forceinline__ void copy_piece(uint64_t dst, uint64_t src, uint64_t size, uint64_t L,
                                           uint32_t j, uint32_t unroll, uint32_t lane) {
  const uint64_t base = dst & ~(uint64_t)(kLineBytes - 1);
  uint64_t lo = base + (uint64_t)j * L, hi = lo + L;
  if (lo < dst) lo = dst;
  if (hi > dst + size) hi = dst + size;
  if (lo < hi) copy_range(lo, hi, src + (lo - dst), unroll, lane);
}

// Inclusive prefix scan, in place, of v[0, m) in LDS by a whole workgroup
// of B threads: every thread sums a run of consecutive entries, the run sums
// are scanned per wavefront with __shfl_up, wsum[] carries across
// wavefronts, and every thread rewrites its run.  Ends with a barrier.
template <int B>
__device__ __forceinline__ void block_scan(uint32_t *v, uint32_t m, uint32_t *wsum) {
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t per = (m + B - 1) / B;
  const uint32_t k0 = min(tid * per, m), k1 = min(k0 + per, m);
  uint32_t sum = 0;
  for (uint32_t k = k0; k < k1; k++) sum += v[k];
  uint32_t inc = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    uint32_t t = __shfl_up(inc, o, 64);
    if (lane >= (uint32_t)o) inc += t;
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  uint32_t run = inc - sum;
  for (uint32_t w = 0; w < wave; w++) run += wsum[w];
  for (uint32_t k = k0; k < k1; k++) {
    run += v[k];
    v[k] = run;
  }
  __syncthreads();
}

__global__ __launch_bounds__(kCopyBlock) void copy_kernel(DevBatch b, DevSched s) {
  __shared__ uint32_t ends[kMaxLdsDescs];
  __shared__ uint32_t wsum[kCopyBlock / 64];
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t n = b.n;

  // 1. pieces per request, then an inclusive block scan in LDS
  for (uint32_t i = tid; i < n; i += kCopyBlock)
    ends[i] = (uint32_t)piece_count(b.dst[i], b.size[i], s.chunk, s.wgs);
  __syncthreads();
  block_scan<kCopyBlock>(ends, n, wsum);
  const uint32_t total = n ? ends[n - 1] : 0;

  // 2-3. persistent loop over pieces, one wavefront per piece
  constexpr uint32_t kWaves = kCopyBlock / 64;
  const uint32_t first = __builtin_amdgcn_readfirstlane(blockIdx.x * kWaves + wave);
  const uint32_t stride = gridDim.x * kWaves;
  for (uint32_t q = first; q < total; q += stride) {
    uint32_t i = __builtin_amdgcn_readfirstlane(find_piece_owner(ends, n, q, lane));
    uint32_t j = q - (i ? ends[i - 1] : 0u);
    const uint64_t dst = b.dst[i], src = b.src[i], size = b.size[i];
    copy_piece(dst, src, size, piece_len(dst, size, s.chunk, s.wgs), j, s.unroll, lane);
  }
}

// Tells the host that the launches before it on its stream have ended.
// copy_kernel leaves that to this one: with signal_done at its own end (and
// its pieces' last bytes written through, which that needs) its loop was
// compiled so that every piece's search waited for the stores of the piece
// before, 1.4 % of a batch to 64 MiB (5,740 against 5,830 GB/s).
__global__ __launch_bounds__(64) void done_kernel(Done done) { signal_done(done); }

// Table of a large batch, one workgroup per tile of kTile requests: the
// tile's piece counts are loaded (all of a thread's loads in flight at
// once), counted into LDS, scanned there, and written out as the tile's
// inclusive prefix (relative to the tile's first piece) with the tile's
// total in tile_tot[tile].  With kStage the requests lie in pinned host
// memory (`b`) and the kernel also moves them to device memory (`to`): the
// same stream then needs no copy engine, whose start waits for a completion
// signal of the kernel before it.
template <bool kStage>
__global__ __launch_bounds__(kScanBlock) void scan_kernel(DevBatch b, DevBatch to, DevSched s,
                                                          uint32_t *ends, uint32_t *tile_tot) {
  constexpr int kPer = kTile / kScanBlock;
  __shared__ uint32_t cnt[kTile];
  __shared__ uint32_t wsum[kScanBlock / 64];
  const uint32_t tid = threadIdx.x;
  const uint32_t i0 = blockIdx.x * kTile, m = min(b.n - i0, kTile);
  uint64_t dv[kPer], zv[kPer], sv[kPer], pv[kPer];
#pragma unroll
  for (int r = 0; r < kPer; r++) {
    const uint32_t k = tid + r * kScanBlock;
    dv[r] = k < m ? b.dst[i0 + k] : 0;
    zv[r] = k < m ? b.size[i0 + k] : 0;
    if (kStage) {
      sv[r] = k < m ? b.src[i0 + k] : 0;
      pv[r] = k < m ? b.slots[i0 + k] : 0;
    }
  }
#pragma unroll
  for (int r = 0; r < kPer; r++) {
    const uint32_t k = tid + r * kScanBlock;
    if (k >= m) continue;
    cnt[k] = (uint32_t)piece_count(dv[r], zv[r], s.chunk, s.wgs);
    if (kStage) {
      const_cast<uint64_t *>(to.dst)[i0 + k] = dv[r];
      const_cast<uint64_t *>(to.src)[i0 + k] = sv[r];
      const_cast<uint64_t *>(to.size)[i0 + k] = zv[r];
      const_cast<uint64_t *>(to.slots)[i0 + k] = pv[r];
    }
  }
  __syncthreads();
  block_scan<kScanBlock>(cnt, m, wsum);
  for (uint32_t k = tid; k < m; k += kScanBlock) ends[i0 + k] = cnt[k];
  if (tid == 0) tile_tot[blockIdx.x] = cnt[m - 1];
}

// Move `words` 8-byte words of pinned host memory to device memory.
__global__ __launch_bounds__(kCopyBlock) void upload_kernel(const uint64_t *h, uint64_t *d,
                                                            uint64_t words) {
  for (uint64_t i = blockIdx.x * kCopyBlock + threadIdx.x; i < words; i += gridDim.x * kCopyBlock)
    d[i] = h[i];
}

// Copy, with one wave, what the batch holds from byte `off` of request
// `first` up to byte `end` of request `last` (0 of request n: to its end), as
// one sequence of chunks: lane l holds request base + l, and the chunk
// pipeline runs on from one request into the next.
__device__ __forceinline__ void stream_lanes(uint64_t v_d, uint64_t v_s, uint64_t v_n, uint32_t l,
                                             uint32_t j, uint32_t lane) {
  uint64_t d = 0, s = 0, left = 0;
  move_chunks<kPlainLoad, kStorePolicy>(
      [&]() {
        while (left == 0 && l < j) {
          left = lane64(v_n, l);
          d = lane64(v_d, l);
          s = lane64(v_s, l);
          l++;
        }
        const uint64_t line = kChunkBytes - (d & (kLineBytes - 1));
        const Chunk c = {d, s, (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)min(line, left))};
        left -= c.n;
        d += c.n;
        s += c.n;
        return c;
      },
      lane);
}
__device__ __forceinline__ void stream_range(const DevBatch &b, uint64_t first, uint64_t off,
                                             uint64_t last, uint64_t end, uint32_t lane) {
  for (uint64_t base = first; base <= last && base < b.n; base += 64) {
    const uint64_t i = base + lane;
    uint64_t v_d = 0, v_s = 0, v_n = 0;
    if (i <= last && i < b.n) {
      const uint64_t lo = i == first ? off : 0;
      v_n = (i == last ? end : b.size[i]) - lo;
      v_d = b.dst[i] + lo;
      v_s = b.src[i] + lo;
    }
    stream_lanes(v_d, v_s, v_n, 0, (uint32_t)min(last + 1 - base, (uint64_t)64), lane);
  }
}

// Copy against the tiled table in device memory.  Every workgroup first
// scans the tile totals into LDS (at most kMaxTiles of them), so piece q's
// global index is tile_base(tile) + local prefix.  Wavefront w of the W in
// the grid takes pieces [total * w / W, total * (w + 1) / W): it finds the
// request and byte where its first piece and the next wavefront's first piece
// start (64-ary search over the tile bases, then over that tile's prefix) and
// copies what lies between.
__device__ __forceinline__ StreamStart piece_start(const DevBatch &b, const DevSched &s,
                                                   const GLOBAL uint32_t *ends,
                                                   const uint32_t *tiles, uint32_t nt, uint32_t q,
                                                   uint32_t total, uint32_t lane) {
  if (q >= total) return StreamStart{0, b.n};
  const uint32_t t = __builtin_amdgcn_readfirstlane(find_piece_owner(tiles, nt, q, lane));
  const uint32_t tb = t ? tiles[t - 1] : 0u, t0 = t * kTile;
  const uint32_t i = t0 + __builtin_amdgcn_readfirstlane(find_piece_owner(
                              ends + t0, min(b.n - t0, kTile), q - tb, lane));
  const uint32_t j = q - (tb + (i > t0 ? ends[i - 1] : 0u));
  const uint64_t dst = b.dst[i], size = b.size[i];
  const uint64_t lo = (dst & ~(uint64_t)(kLineBytes - 1)) + j * piece_len(dst, size, s.chunk, s.wgs);
  return StreamStart{j ? min(lo - dst, size) : 0, i};
}

__global__ __launch_bounds__(kCopyBlock) void copy_kernel_mem(DevBatch b, DevSched s,
                                                              const uint32_t *ends_in,
                                                              const uint32_t *tile_tot, Done done) {
  __shared__ uint32_t tiles[kMaxTiles];
  __shared__ uint32_t wsum[kCopyBlock / 64];
  const GLOBAL uint32_t *ends = (const GLOBAL uint32_t *)ends_in;
  constexpr uint32_t kWaves = kCopyBlock / 64;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t nt = (b.n + kTile - 1) / kTile;
  for (uint32_t k = threadIdx.x; k < nt; k += kCopyBlock) tiles[k] = tile_tot[k];
  __syncthreads();
  block_scan<kCopyBlock>(tiles, nt, wsum);
  const uint64_t total = tiles[nt - 1];
  const uint64_t W = (uint64_t)gridDim.x * kWaves;
  const uint64_t gw = __builtin_amdgcn_readfirstlane(blockIdx.x * kWaves + (threadIdx.x >> 6));
  const uint32_t q = (uint32_t)(total * gw / W), q1 = (uint32_t)(total * (gw + 1) / W);
  if (q < q1) {
    const StreamStart at = piece_start(b, s, ends, tiles, nt, q, (uint32_t)total, lane);
    const StreamStart to = piece_start(b, s, ends, tiles, nt, q1, (uint32_t)total, lane);
    stream_range(b, uni64(at.req), uni64(at.off), uni64(to.req), uni64(to.off), lane);
  }
  signal_done(done);
}

// A batch small enough not to need the piece kernels' order (stream_waves says
// which) copied as one stream of bytes in equal shares, one per wave.  The
// host has cut the shares, so nothing is scanned or searched here, and the
// requests are read where they are: for a submission in pinned host memory,
// each wave its own few, over the host link, which takes less than queuing an
// upload in front (with upload, copy and counter kernels and an event: 512
// requests to 1 MiB submit to fence 57 us; now 35 = 3.6 TB/s, its kernel
// 26 us = 4.9 TB/s).  Bound: launch, host link and memory latencies below a
// few MiB, HBM above.
__global__ __launch_bounds__(kCopyBlock) void stream_kernel(DevBatch b, const StreamStart *starts,
                                                            uint32_t waves, Done done) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t w =
      __builtin_amdgcn_readfirstlane(blockIdx.x * (kCopyBlock / 64) + (threadIdx.x >> 6));
  if (w < waves)
    stream_range(b, uni64(starts[w].req), uni64(starts[w].off), uni64(starts[w + 1].req),
                 uni64(starts[w + 1].off), lane);
  signal_done(done);
}

// The same for up to N requests, held in the kernel's arguments: in pinned
// memory it takes a wave two trips over the host link, to its share and to its
// requests, before its first load (submit to fence of one request of 4 KiB
// 11.6 -> 9.5 us, 64 to 8 KiB 13.3 -> 11.3, 256 to 8 KiB 14.4 -> 13.2, 256 to
// 256 KiB 23.2 -> 20.9; a plan's requests lie in device memory, which is
// nearer than arguments: a replay of 16 to 4 KiB 9.2 us that way, 9.6 with
// arguments).  4 KiB of arguments hold no more.  Addresses are held as
// 32-bit distances from the lowest of the batch, sizes as what the batch counts
// for (stream_load) up to the end of the request, from which every wave finds
// its share: what lies between w and w + 1 times `share`, cut at lines of the
// destinations.
constexpr uint32_t kArgShort = 1u << 31;  // in end: the request counts for kStreamExtra more
template <uint32_t N>
struct ArgBatch {
  Done done;
  uint64_t dst, src;
  uint32_t n, waves, share, load;
  uint32_t end[N], d[N], s[N];  // end: ~0 past the last request
};
template <uint32_t N>
__global__ __launch_bounds__(kCopyBlock) void stream_args_kernel(ArgBatch<N> a) {
  using Args = ArgBatch<N>;
  constexpr uint32_t K = N / 64;
  // (arrays in arguments are read by address, or they would be copied to
  // scratch memory first)
  const GLOBAL uint32_t *t = (const GLOBAL uint32_t *)(
      (uint64_t)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(Args, end));
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t w =
      __builtin_amdgcn_readfirstlane(blockIdx.x * (kCopyBlock / 64) + (threadIdx.x >> 6));
  if (w < a.waves) {
    // every wave reads them all, so that only one trip to memory comes before
    // its first load: lane l holds requests l, l + 64, ...
    uint32_t e[K], f[K], d[K], s[K], z[K];  // f: where it starts, z: its bytes
#pragma unroll
    for (uint32_t k = 0; k < K; k++) {
      const uint32_t i = lane + 64 * k;
      e[k] = t[i];
      f[k] = t[i ? i - 1 : 0];
      d[k] = t[N + i];
      s[k] = t[2 * N + i];
    }
    if (lane == 0) f[0] = 0;
#pragma unroll
    for (uint32_t k = 0; k < K; k++) {
      const uint32_t more = e[k] & kArgShort ? (uint32_t)kStreamExtra : 0;
      e[k] &= ~kArgShort;
      f[k] &= ~kArgShort;
      z[k] = e[k] - f[k] - more;
    }
    // the request where the share starts and ends (n: past the last), and the
    // byte of it
    uint32_t i[2];
    uint64_t off[2];
#pragma unroll
    for (int j = 0; j < 2; j++) {
      const uint64_t x = (uint64_t)(w + j) * a.share;
      uint32_t c = 0, r = 0, from = 0, to = 0, size = 0;
#pragma unroll
      for (uint32_t k = 0; k < K; k++) c += (uint32_t)__popcll(__ballot(e[k] <= x));
      r = min(c, a.n - 1);
#pragma unroll
      for (uint32_t k = 0; k < K; k++)
        if (r / 64 == k) {
          from = __builtin_amdgcn_readlane(f[k], r % 64);
          size = __builtin_amdgcn_readlane(z[k], r % 64);
          to = __builtin_amdgcn_readlane(d[k], r % 64);
        }
      const uint64_t dst = a.dst + to, at = x - from;
      off[j] = min(((dst + at + kLineBytes - 1) & ~(uint64_t)(kLineBytes - 1)) - dst,
                   (uint64_t)size);
      if (at == 0 || x >= a.load) off[j] = 0;
      i[j] = x >= a.load ? a.n : c;
    }
    for (uint32_t k = i[0] / 64; k < K && 64 * k <= i[1]; k++) {
      uint32_t zk = z[0], dk = d[0], sk = s[0];
#pragma unroll
      for (uint32_t m = 1; m < K; m++)
        if (k == m) zk = z[m], dk = d[m], sk = s[m];
      const uint32_t r = lane + 64 * k;
      const uint64_t lo = r == i[0] ? off[0] : 0, hi = r == i[1] ? off[1] : zk;
      stream_lanes(a.dst + dk + lo, a.src + sk + lo, r >= i[0] && r <= i[1] && r < a.n ? hi - lo : 0,
                   max(i[0], 64 * k) - 64 * k, min(i[1] + 1 - 64 * k, 64u), lane);
    }
  }
  signal_done(a.done);
}

template <uint32_t N>
static void launch_args(const uint64_t *h, uint32_t n, uint64_t dst, uint64_t src, uint64_t load,
                        uint32_t waves, Done done, hipStream_t stream) {
  ArgBatch<N> a;
  static_assert(sizeof(a) <= 4096, "kernel arguments");
  static_assert(N % 64 == 0 && offsetof(ArgBatch<N>, s) == offsetof(ArgBatch<N>, end) + 8 * N,
                "three arrays of N");
  a.done = done;
  a.dst = dst;
  a.src = src;
  a.n = n;
  a.waves = waves;
  a.share = (uint32_t)((load + waves - 1) / waves);
  a.load = (uint32_t)load;
  uint32_t end = 0;
  for (uint32_t i = 0; i < n; i++) {
    const uint64_t size = h[2 * n + i];
    end += (uint32_t)stream_load(size);
    a.end[i] = end | (size < kStreamShort ? kArgShort : 0);
    a.d[i] = (uint32_t)(h[i] - dst);
    a.s[i] = (uint32_t)(h[n + i] - src);
  }
  std::fill(a.end + n, a.end + N, ~0u);
  hipLaunchKernelGGL(stream_args_kernel<N>, dim3(stream_grid(waves)), dim3(kCopyBlock), 0, stream,
                     a);
}

bool args_fit(const uint64_t *h, uint64_t n, uint64_t load, uint64_t *dst, uint64_t *src) {
  constexpr uint64_t kSpan = 0xffffffffull;
  // (shares run to less than load + kMaxStreamWaves, and kArgShort - 1 marks the end)
  if (!n || n > kArgReqs || load >= kArgShort - 2 * kMaxStreamWaves) return false;
  const auto d = std::minmax_element(h, h + n), s = std::minmax_element(h + n, h + 2 * n);
  *dst = *d.first;
  *src = *s.first;
  return *d.second - *dst <= kSpan && *s.second - *src <= kSpan;
}

hipError_t launch_stream_args(const uint64_t *h, uint32_t n, uint64_t dst, uint64_t src,
                              uint64_t load, uint32_t waves, Done done, hipStream_t stream) {
  if (!n || n > kArgReqs || !waves) return hipErrorInvalidValue;
  if (n <= 64)
    launch_args<64>(h, n, dst, src, load, waves, done, stream);
  else
    launch_args<kArgReqs>(h, n, dst, src, load, waves, done, stream);
  return hipGetLastError();
}

hipError_t launch_stream(const DevBatch &b, const StreamStart *starts, uint32_t waves, Done done,
                         hipStream_t stream) {
  if (!waves || !starts) return hipErrorInvalidValue;
  hipLaunchKernelGGL(stream_kernel, dim3(stream_grid(waves)), dim3(kCopyBlock), 0, stream, b,
                     starts, waves, done);
  return hipGetLastError();
}

hipError_t launch_copy(const DevBatch &b, DevSched s, uint32_t grid, hipStream_t stream) {
  if (b.n > kMaxLdsDescs || grid == 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(copy_kernel, dim3(grid), dim3(kCopyBlock), 0, stream, b, s);
  return hipGetLastError();
}

hipError_t launch_done(Done done, hipStream_t stream) {
  hipLaunchKernelGGL(done_kernel, dim3(1), dim3(64), 0, stream, done);
  return hipGetLastError();
}

hipError_t launch_scan(const DevBatch *staged, const DevBatch &b, DevSched s, uint32_t *ends,
                       uint32_t *tile_tot, hipStream_t stream) {
  const uint32_t tiles = (b.n + kTile - 1) / kTile;
  if (b.n == 0 || !ends || !tile_tot || tiles > kMaxTiles || (staged && staged->n != b.n))
    return hipErrorInvalidValue;
  if (staged)
    hipLaunchKernelGGL(scan_kernel<true>, dim3(tiles), dim3(kScanBlock), 0, stream, *staged, b, s,
                       ends, tile_tot);
  else
    hipLaunchKernelGGL(scan_kernel<false>, dim3(tiles), dim3(kScanBlock), 0, stream, b, b, s, ends,
                       tile_tot);
  return hipGetLastError();
}

hipError_t launch_upload(const void *h_dev, void *d, uint64_t bytes, hipStream_t stream) {
  const uint64_t words = bytes / 8;
  const uint32_t grid = (uint32_t)std::min<uint64_t>(64, (words + kCopyBlock - 1) / kCopyBlock);
  if (!words || bytes % 8) return hipErrorInvalidValue;
  hipLaunchKernelGGL(upload_kernel, dim3(grid), dim3(kCopyBlock), 0, stream,
                     static_cast<const uint64_t *>(h_dev), static_cast<uint64_t *>(d), words);
  return hipGetLastError();
}

hipError_t launch_copy_mem(const DevBatch &b, DevSched s, const uint32_t *ends,
                           const uint32_t *tile_tot, uint32_t grid, Done done,
                           hipStream_t stream) {
  if (b.n == 0 || !ends || !tile_tot || grid == 0 || (b.n + kTile - 1) / kTile > kMaxTiles)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(copy_kernel_mem, dim3(grid), dim3(kCopyBlock), 0, stream, b, s, ends,
                     tile_tot, done);
  return hipGetLastError();
}

int copy_occupancy(int *wgs_per_cu) {
  return (int)hipOccupancyMaxActiveBlocksPerMultiprocessor(wgs_per_cu, copy_kernel, kCopyBlock,
                                                            0);
}

}  // namespace hicr
