// Host driver for how stream_kernel's rule counts short requests
// (paper_2509_01425_amd/csrc/stream_plan.h): reads cases "n_cu n" followed by n lines
// "dst size" from stdin and prints "waves" and, when it is not 0, "off req" of
// every start, one line per case.
#include <cstdio>
#include <vector>

#include "stream_plan.h"

int main() {
  unsigned long long cu, n, a, b;
  while (std::scanf("%llu %llu", &cu, &n) == 2) {
    std::vector<uint64_t> dst(n), size(n);
    uint64_t bytes = 0, n_short = 0;
    for (uint64_t i = 0; i < n; i++) {
      if (std::scanf("%llu %llu", &a, &b) != 2) return 1;
      dst[i] = a;
      size[i] = b;
      bytes += b;
      n_short += b < hicr::kStreamShort;
    }
    const uint32_t w = hicr::stream_waves(n, bytes, cu, 0, n_short);
    std::printf("%u", w);
    if (w) {
      std::vector<hicr::StreamStart> s(w + 1);
      hicr::stream_starts(dst.data(), size.data(), n, bytes, w, 128, s.data(), n_short);
      for (const auto &x : s) std::printf(" %llu %llu", (unsigned long long)x.off, (unsigned long long)x.req);
    }
    std::printf("\n");
  }
  return 0;
}
