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
inline uint32_t stream_waves(uint64_t n, uint64_t bytes, uint64_t n_cu, uint64_t per_cu) {
  if (n > kStreamMaxReqs || bytes > kStreamMaxBytes + n * kStreamPerReq) return 0;
  const uint64_t most = std::min<uint64_t>(kMaxStreamWaves, n_cu * (per_cu ? per_cu : 1) * 4);
  return (uint32_t)std::min(most, std::max<uint64_t>(1, (bytes + kStreamShare - 1) / kStreamShare));
}

// Equal shares of the batch's bytes, cut at `line`-byte lines (a power of two)
// of the destinations: wave w copies what lies between out[w] and out[w + 1]
// (out[waves] is the end of the batch).  A division per wave would cost 2 us of
// host time for 1,024 waves.
inline void stream_starts(const uint64_t *dst, const uint64_t *size, uint64_t n, uint64_t bytes,
                          uint32_t waves, uint64_t line, StreamStart *out) {
  const uint64_t share = bytes / waves, rest = bytes % waves;
  uint64_t i = 0, before = 0;  // bytes of the requests before i
  uint64_t at = 0, part = 0;   // bytes * w / waves, and the remainder
  for (uint32_t w = 0; w < waves; w++) {
    while (i < n && before + size[i] <= at) before += size[i++];
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

}  // namespace hicr
