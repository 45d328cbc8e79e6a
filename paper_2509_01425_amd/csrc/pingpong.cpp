// pingpong.cpp -- host side of the two-endpoint ping-pong (the paper's Test
// Case 1 on one GPU).
#include <algorithm>

#include "pingpong.h"
#include "runtime.h"

using namespace hicr;

constexpr size_t kGroupWords = 1 << 18;  // at most 2 MiB of words for several sizes together

extern "C" {

int hicr_pingpong(hicr_ctx c, hicr_slot src, hicr_slot dst, hicr_slot ring_a, hicr_slot ring_b,
                  hicr_slot buf, const uint64_t *sizes, uint32_t n_sizes, uint32_t reps,
                  uint32_t wgs_per_endpoint, uint64_t *rtt_ticks) {
  return guarded([&]() -> int {
    if (!c || (n_sizes && (!sizes || !rtt_ticks)) || reps == 0 || reps > 100000) return HICR_EINVAL;
    std::lock_guard<std::mutex> g(c->mu);
    (void)hipSetDevice(c->device);
    uint64_t smax = 0;
    for (uint32_t i = 0; i < n_sizes; i++) smax = std::max(smax, sizes[i]);
    const hicr_slot ids[5] = {src, dst, ring_a, ring_b, buf};
    uint64_t base[5];
    for (int i = 0; i < 5; i++) {
      if (ids[i] >= c->slots.size() || !c->slots[ids[i]].live) return fail(c, HICR_EBADSLOT, "slot");
      const Slot &s = c->slots[ids[i]];
      if (s.space != HICR_MEM_HBM) return fail(c, HICR_EUNSUPPORTED, "slot not in HBM");
      if (s.base % 16) return fail(c, HICR_EINVAL, "slots must be 16-byte aligned");
      if (s.size < smax) return fail(c, HICR_ERANGE, "slot smaller than the largest message");
      base[i] = s.base;
    }
    int occ = 0;
    if (pingpong_occupancy(&occ) != 0 || occ < 1) occ = 1;
    const uint64_t cap = (uint64_t)c->n_cu * occ / 2;
    int rc = flush_pending(c);
    if (rc == HICR_OK) rc = wait_all(c);
    if (rc != HICR_OK) return rc;
    // a workgroup for every 16 KiB of message, its four waves' chunks in
    // flight at once (one-way 64 KiB 3.0 us, with 32 KiB each 3.1, 64 KiB each
    // 4.7; 4 MiB 5.9, 5.4, 6.4; more than 256 of them: 16 MiB 11.2 us, not 10.2)
    auto workgroups = [&](uint64_t size) {
      uint64_t W = wgs_per_endpoint;
      if (W == 0) W = std::max<uint64_t>(1, std::min<uint64_t>(256, size >> 14));
      return (uint32_t)std::min<uint64_t>(W, cap);
    };
    // The sizes are launched one behind the other, as many at a time as fit
    // the word buffer: a line with the error word, then per size its counter
    // lines and the two clock readings of every round trip.
    auto words_of = [&](uint64_t size) {
      const size_t w = pingpong_words(workgroups(size)) + 2 * (size_t)reps;
      return (w + kLineWords - 1) / kLineWords * kLineWords;
    };
    size_t all = kLineWords, words = 0;
    for (uint32_t i = 0; i < n_sizes; i++) {
      all += words_of(sizes[i]);
      words = std::max(words, kLineWords + words_of(sizes[i]));
    }
    words = std::max(words, std::min(all, kGroupWords));
    if (words > c->pp_words) {
      if (c->pp_d) (void)hipFree(c->pp_d);
      if (c->pp_h) (void)hipHostFree(c->pp_h);
      c->pp_d = c->pp_h = nullptr;
      c->pp_words = 0;
      void *dv = nullptr, *hv = nullptr;
      if (hipMalloc(&dv, words * 8) != hipSuccess) return fail(c, HICR_ENOMEM, "ping-pong words");
      c->pp_d = static_cast<uint64_t *>(dv);
      if (hipHostMalloc(&hv, words * 8, hipHostMallocDefault) != hipSuccess)
        return fail(c, HICR_ENOMEM, "ping-pong words");
      c->pp_h = static_cast<uint64_t *>(hv);
      c->pp_words = words;
    }
    uint64_t *d = c->pp_d, *h = c->pp_h;
    for (uint32_t i0 = 0; i0 < n_sizes && rc == HICR_OK;) {
      size_t used = kLineWords;
      uint32_t i1 = i0;
      while (i1 < n_sizes && used + words_of(sizes[i1]) <= c->pp_words) used += words_of(sizes[i1++]);
      hipError_t e = hipMemsetAsync(d, 0, used * 8, c->stream);
      size_t at = kLineWords;
      for (uint32_t i = i0; i < i1 && e == hipSuccess; i++) {
        PingPongArgs a;
        a.src = base[0];
        a.dst = base[1];
        a.ring_a = base[2];
        a.ring_b = base[3];
        a.buf = base[4];
        a.size = sizes[i];
        a.W = workgroups(sizes[i]);
        a.reps = reps;
        a.ctr = d + at;
        a.t_start = a.ctr + pingpong_words(a.W);
        a.t_end = a.t_start + reps;
        a.err = reinterpret_cast<uint32_t *>(d);
        a.timeout_ticks = 1'000'000'000ull;  // 10 s without progress
        e = launch_pingpong(a, c->stream);
        at += words_of(sizes[i]);
      }
      if (e == hipSuccess) e = hipMemcpyAsync(h, d, used * 8, hipMemcpyDeviceToHost, c->stream);
      if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
      if (e != hipSuccess) {
        rc = hip_fail(c, e, "ping-pong");
        break;
      }
      at = kLineWords;
      for (uint32_t i = i0; i < i1; i++) {
        const uint64_t *t = h + at + pingpong_words(workgroups(sizes[i]));
        at += words_of(sizes[i]);
        if (h[0] && t[2 * (size_t)reps - 1] == 0) {  // the first size that did not end
          rc = fail(c, HICR_ETIMEDOUT, "ping-pong of %llu bytes made no progress",
                    (unsigned long long)sizes[i]);
          break;
        }
        for (uint32_t k = 0; k < reps; k++) rtt_ticks[(size_t)i * reps + k] = t[reps + k] - t[k];
      }
      i0 = i1;
    }
    return rc;
  });
}

}  // extern "C"
