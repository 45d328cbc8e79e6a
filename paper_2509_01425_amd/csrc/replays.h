// replays.h -- which replays of a plan have ended, from its done words.  Kept
// free of HIP so that it can be tested on the host.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

namespace hicr {

// Replays are numbered in the order in which they run, one after another, and
// each raises the first few of the plan's words to its number when it ends:
// as many as its launch has workgroups, so another number of them once the copy
// grid has been set anew.  Words that an earlier replay did not raise say
// nothing about it; so the numbers of words are remembered while replays that
// had them may be in flight.
class Replays {
 public:
  // Replay `seq`, which raises `words` words, has been queued; idle: every
  // earlier one is known to have ended.
  void queued(uint64_t seq, uint32_t words, bool idle) {
    if (idle) runs_.clear();
    if (runs_.empty() || runs_.back().words != words) runs_.push_back(Run{seq, words});
  }
  // The number of the last replay that has ended (0: none).
  uint64_t ended(const uint64_t *w) const {
    uint64_t last = ~0ull;  // of the run looked at
    for (size_t k = runs_.size(); k-- > 0; last = runs_[k].first - 1) {
      uint64_t done = last;
      for (uint32_t i = 0; i < runs_[k].words; i++)
        done = std::min(done, __atomic_load_n(&w[i], __ATOMIC_ACQUIRE));
      if (done >= runs_[k].first) return done;
    }
    return last == ~0ull ? 0 : last;
  }

 private:
  struct Run {
    uint64_t first;  // replay
    uint32_t words;
  };
  std::vector<Run> runs_;
};

}  // namespace hicr
