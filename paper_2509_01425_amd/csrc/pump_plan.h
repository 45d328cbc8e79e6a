// pump_plan.h -- which endpoints of a channel pump are whole workgroups.
//
// A pump's workgroups must all be resident at once.  This is the rule that
// shares the `cap` workgroups a device holds among the producers (one per
// stream), the consumers of single-producer rings and the teams that drain
// locking rings, kept free of HIP so that it can be tested on the host.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

namespace hicr {

struct PumpPlan {
  bool fits = false;
  uint64_t need = 0;           // workgroups of the smallest form
  bool lock_groups = false;    // a locking ring's producers are workgroups, not waves
  bool ind_groups = false;     // so are the other producers and their consumers
  std::vector<uint32_t> team;  // workgroups that drain each locking ring
  uint64_t ind_units = 0;      // consumers of the other rings
  uint32_t split = 1;          // workgroups of each of their ends,
  uint32_t share = 1;          // this many to a team that shares a group of messages
  uint64_t wgs = 0;            // workgroups in all
};

// cap workgroups, on n_cu compute units; n_lock producers on locking rings that want teams of `want`
// workgroups (at least 1 each), n_ind producers on rings of their own; a
// consumer holds at most `max_rings` rings; an end of a ring of its own may
// be split over `max_split` workgroups.
//
// Groups or waves.  A producer that is one wave has 8 KiB in flight, so a few
// streams are bound by it (serving 16 bursts of up to 256 messages to
// 256 KiB: 1.38 ms with waves, 0.87 with groups), while many streams fill the
// memory either way.  A locking ring's producers come first, since each batch
// of theirs holds up the ones behind it (64 rings of 8 beside 1,024 SPSC
// streams: 5.43 ms a pass with waves, 5.10 with groups), as long as every
// locking ring keeps a team of two; then, if all of it fits, the other
// producers and consumers.  Rings share a consumer wave only when there are
// more of them than waves.
//
// Splits.  One compute unit copies 20-26 GB/s however many waves it runs (a
// pump of 16 such bursts took 471 us with blocks of 256 threads, 497 with
// 1,024), so while a pump leaves compute units unused both ends of its rings
// are split: those 16 bursts 509 -> 203 us, two streams 454 -> 175, 60 streams
// (split in two) 540 -> 398, 16 streams of 4,096 messages to 64 B 1,570 -> 875;
// 100 streams are as before (640).  From four workgroups on two share each
// group of messages, since the largest message otherwise sets the time of its
// turn (16 bursts: 1 workgroup to a group 256 us, 2: 207, 4: 248).  One
// workgroup per compute unit is the limit, which leaves other pumps room
// beside this one.
inline PumpPlan plan_endpoints(uint64_t cap, uint64_t n_lock, uint64_t n_ind,
                               const std::vector<uint64_t> &want, uint64_t max_rings,
                               uint64_t n_cu = 0, uint64_t max_split = 1) {
  PumpPlan p;
  const uint64_t prod = (n_lock + n_ind + 3) / 4, rings = want.size();
  const uint64_t min_units = (n_ind + max_rings - 1) / max_rings;
  p.need = prod + rings + min_units;
  if (p.need > cap) return p;
  p.fits = true;
  // teams as wanted, the largest trimmed while the rest would not fit
  uint64_t total = 0;
  for (uint64_t t : want) {
    p.team.push_back((uint32_t)std::max<uint64_t>(1, t));
    total += p.team.back();
  }
  while (prod + total + min_units > cap) {
    --*std::max_element(p.team.begin(), p.team.end());
    total--;
  }
  const uint64_t ind_wave_wgs = (n_ind + 3) / 4;
  const uint64_t lock_first = n_lock + 2 * ind_wave_wgs;
  if (rings && lock_first + 2 * rings <= cap) {
    p.lock_groups = true;
    const uint32_t most = (uint32_t)std::min<uint64_t>(~0u, (cap - lock_first) / rings);
    total = 0;
    for (uint32_t &t : p.team) total += t = std::min(t, most);
  }
  p.ind_groups = (p.lock_groups || !rings) && n_lock + 2 * n_ind + total <= cap;
  // producers that are all waves share workgroups
  const uint64_t prod_wgs = p.ind_groups    ? n_lock + n_ind
                            : p.lock_groups ? n_lock + ind_wave_wgs
                                            : prod;
  p.ind_units = p.ind_groups ? n_ind : std::min(n_ind, 4 * (cap - prod_wgs - total));
  p.wgs = prod_wgs + total + (p.ind_groups ? n_ind : (p.ind_units + 3) / 4);
  const uint64_t room = std::min(cap, n_cu);
  if (p.ind_groups && n_ind && max_split > 1 && p.wgs < room) {
    p.split = (uint32_t)std::min(max_split, (room - n_lock - total) / (2 * n_ind));
    if (p.split >= 4) p.share = 2;
    p.split -= p.split % p.share;
    p.wgs += 2 * n_ind * (p.split - 1);
  }
  return p;
}

}  // namespace hicr
