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
  uint64_t wgs = 0;            // workgroups in all
};

// cap workgroups; n_lock producers on locking rings that want teams of `want`
// workgroups (at least 1 each), n_ind producers on rings of their own; a
// consumer holds at most `max_rings` rings.
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
inline PumpPlan plan_endpoints(uint64_t cap, uint64_t n_lock, uint64_t n_ind,
                               const std::vector<uint64_t> &want, uint64_t max_rings) {
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
  return p;
}

}  // namespace hicr
