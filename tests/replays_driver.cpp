// Host driver for the count of ended replays (paper_2509_01425_amd/csrc/replays.h).
// Reads "q words idle" (the next replay is queued), "r word value" (a word is
// raised) and "e" (print how many replays have ended) from stdin.
#include <cstdio>

#include "replays.h"

int main() {
  hicr::Replays r;
  uint64_t w[64] = {}, seq = 0;
  unsigned long long a, b;
  char op;
  while (std::scanf(" %c", &op) == 1) {
    if (op == 'q' && std::scanf("%llu %llu", &a, &b) == 2)
      r.queued(++seq, (uint32_t)a, b != 0);
    else if (op == 'r' && std::scanf("%llu %llu", &a, &b) == 2)
      w[a] = b;
    else if (op == 'e')
      std::printf("%llu\n", (unsigned long long)r.ended(w));
    else
      return 1;
  }
  return 0;
}
