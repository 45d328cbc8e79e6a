// Host driver for stream_kernel's sharing rule (paper_2509_01425_amd/csrc/stream_plan.h):
// reads cases "n_cu per_cu n" followed by n lines "dst size" from stdin and prints
// "waves" and, when it is not 0, "off req" of every start, one line per case.
#include <cstdio>
#include <vector>

#include "stream_plan.h"

int main() {
  unsigned long long cu, pc, n, a, b;
  while (std::scanf("%llu %llu %llu", &cu, &pc, &n) == 3) {
    std::vector<uint64_t> dst(n), size(n);
    uint64_t bytes = 0;
    for (uint64_t i = 0; i < n; i++) {
      if (std::scanf("%llu %llu", &a, &b) != 2) return 1;
      dst[i] = a;
      size[i] = b;
      bytes += b;
    }
    const uint32_t w = hicr::stream_waves(n, bytes, cu, pc);
    std::printf("%u", w);
    if (w) {
      std::vector<hicr::StreamStart> s(w + 1);
      hicr::stream_starts(dst.data(), size.data(), n, bytes, w, 128, s.data());
      for (const auto &x : s) std::printf(" %llu %llu", (unsigned long long)x.off, (unsigned long long)x.req);
    }
    std::printf("\n");
  }
  return 0;
}
