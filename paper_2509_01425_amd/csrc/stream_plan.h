// stream_plan.h -- how a batch is shared among the waves of stream_kernel.
// Kept free of HIP so that it can be tested on the host.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace hicr {

// Where a wave of stream_kernel starts: byte `off` of request `req`.
struct StreamStart {
  uint64_t off;
  uint64_t req;
};

constexpr uint32_t kMaxStreamWaves = 4096;    // of one launch
constexpr uint64_t kStreamMaxReqs = 4096;
constexpr uint64_t kStreamShare = 4096;       // fewest bytes worth a wave
constexpr uint64_t kStreamMaxBytes = 256ull << 20;
constexpr uint64_t kStreamPerReq = 160 << 10;

// Bytes up to which a batch of n requests is one for the stream kernel under a
// schedule of `chunk`-byte pieces.  Pieces of 4 KiB keep a batch of a few hundred
// MiB together best, and so are preferred earlier (stream against pieces of 4
// and of 64 KiB, us: 16 requests of 160 MiB in all 75 / 74 / 79, of 192 MiB 89 /
// 85 / 91, of 256 MiB 119 / 111 / 118; 256 requests of 192 MiB 94 / 94 / 104, of
// 224 MiB 107 / 107 / 111; 1,024 of 256 MiB 127 / 130 / 133).
constexpr uint32_t kStreamSmallPiece = 4 << 10;
inline uint64_t stream_most(uint64_t n, uint32_t chunk) {
  return (chunk <= kStreamSmallPiece ? 160ull << 20 : kStreamMaxBytes) + n * kStreamPerReq;
}

// A request costs a wave a step of its own however short it is, and a run of
// short ones must not be left to one wave: so a request below kStreamShort
// bytes counts for kStreamExtra more wherever a batch is shared out, which
// leaves a wave at most two of them while there are waves left.  (Shared by
// bytes alone 4,096 requests of 1 B took 1,100 us and 256 of them 74, now 27
// and 13; four to a wave cost 256 of them 1 us, one to a wave 1,024 of them 1.)
constexpr uint64_t kStreamShort = 1024, kStreamExtra = 2048;
inline uint64_t stream_load(uint64_t size) { return size + (size < kStreamShort ? kStreamExtra : 0); }

// Waves that copy a batch of n requests and `bytes` bytes as one stream on a
// device of n_cu units (per_cu workgroups of four waves each, 0: one); 0 when
// the batch is one for the piece kernels.  One workgroup per CU is the
// fastest at every size (64 MiB in 512 requests 35.3 us, with two 37.5, with
// four 45.3); half the share costs a single 16 KiB request 1 us, twice the
// share changes nothing.
//
// Where the line lies (three states in turn; stream against pieces): 512
// requests to 64 KiB 18 against 26 us, to 1 MiB 35 / 56, to 4 MiB (240 MiB)
// 107 / 112; 64 requests of 4 MiB 118 / 125, of 6 MiB 180 / 175, of 12 MiB
// 347 / 312: past 256 MiB the piece kernels' order, in which all waves sweep
// the batch together, gains ~0.07 us per MiB.  They also take ~11 ns a
// request more (upload, a scan of the batch in every workgroup, a search per
// piece): 4,096 requests of 276 MiB 140 / 184, of 1.7 GiB 759 / 700.
//
// n_short: how many of the requests are short (0: none, or count them by their
// bytes all the same).  link: most of the bytes are read from host memory.  The
// host link is full with few waves, and reads longer runs faster: no more than
// kLinkWaves, or one for kLinkShare bytes or for two short requests (4 MiB 84 us
// with 64 waves, 91 with 256, 107 with 1,024; 16 MiB 315 and 352).
constexpr uint64_t kLinkWaves = 64, kLinkShare = 64 << 10;
inline uint32_t stream_waves(uint64_t n, uint64_t bytes, uint64_t n_cu, uint64_t per_cu,
                             uint64_t n_short = 0, bool link = false) {
  if (n > kStreamMaxReqs || bytes > kStreamMaxBytes + n * kStreamPerReq) return 0;
  uint64_t most = std::min<uint64_t>(kMaxStreamWaves, n_cu * (per_cu ? per_cu : 1) * 4);
  if (link) most = std::min(most, std::max({kLinkWaves, bytes / kLinkShare, n_short / 2}));
  const uint64_t load = bytes + n_short * kStreamExtra;
  return (uint32_t)std::min(most, std::max<uint64_t>(1, (load + kStreamShare - 1) / kStreamShare));
}

// Equal shares of what the batch counts for, its bytes and the extra for each
// of its n_short short requests, cut at `line`-byte lines (a power of two)
// of the destinations: wave w copies what lies between out[w] and out[w + 1]
// (out[waves] is the end of the batch).  With n_short = 0 every request counts
// as its bytes.  A division per wave would cost 2 us of host time for 1,024
// waves.
template <class Load>
inline void stream_cut(const uint64_t *dst, const uint64_t *size, uint64_t n, uint64_t load,
                       uint32_t waves, uint64_t line, StreamStart *out, Load of) {
  const uint64_t share = load / waves, rest = load % waves;
  uint64_t i = 0, before = 0, next = n ? of(size[0]) : ~0ull;  // load before i, and before i + 1
  uint64_t at = 0, part = 0;  // load * w / waves, and the remainder
  for (uint32_t w = 0; w < waves; w++) {
    while (next <= at) {
      before = next;
      next = ++i < n ? next + of(size[i]) : ~0ull;
    }
    uint64_t off = i < n ? at - before : 0;
    if (off) off = std::min(((dst[i] + off + line - 1) & ~(line - 1)) - dst[i], size[i]);
    out[w] = StreamStart{off, i};
    at += share;
    part += rest;
    if (part >= waves) {
      part -= waves;
      at++;
    }
  }
  out[waves] = StreamStart{0, n};
}
inline void stream_starts(const uint64_t *dst, const uint64_t *size, uint64_t n, uint64_t bytes,
                          uint32_t waves, uint64_t line, StreamStart *out, uint64_t n_short = 0) {
  if (n_short)
    stream_cut(dst, size, n, bytes + n_short * kStreamExtra, waves, line, out, stream_load);
  else
    stream_cut(dst, size, n, bytes, waves, line, out, [](uint64_t z) { return z; });
}

}  // namespace hicr
