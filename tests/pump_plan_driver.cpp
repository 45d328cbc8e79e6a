// Host driver for the pump's endpoint rule (paper_2509_01425_amd/csrc/pump_plan.h):
// reads cases "cap n_lock n_ind max_rings n_cu max_split n_want want..." from
// stdin and prints "fits need lock_groups ind_groups ind_units wgs split share
// n_team team..." per case.
#include <cstdio>
#include <vector>

#include "pump_plan.h"

int main() {
  unsigned long long cap, nl, ni, mr, cu, ms, nw, w;
  while (std::scanf("%llu %llu %llu %llu %llu %llu %llu", &cap, &nl, &ni, &mr, &cu, &ms, &nw) == 7) {
    std::vector<uint64_t> want(nw);
    for (auto &x : want) {
      if (std::scanf("%llu", &w) != 1) return 1;
      x = w;
    }
    const hicr::PumpPlan p = hicr::plan_endpoints(cap, nl, ni, want, mr, cu, ms);
    std::printf("%d %llu %d %d %llu %llu %u %u %zu", p.fits, (unsigned long long)p.need, p.lock_groups,
                p.ind_groups, (unsigned long long)p.ind_units, (unsigned long long)p.wgs,
                p.split, p.share, p.team.size());
    for (uint32_t t : p.team) std::printf(" %u", t);
    std::printf("\n");
  }
  return 0;
}
