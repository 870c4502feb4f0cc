// The shares of a batched launch on the host.  Reads "items grid cost lgs"
// rows; prints share, the items' waves with work and "1" when the parts of an
// item cover its blocks once, in order.
#include <cstdio>

#include "rlx_share.hpp"

int main() {
  unsigned items, grid, cost, lgs;
  while (std::scanf("%u %u %u %u", &items, &grid, &cost, &lgs) == 4) {
    const uint32_t share = rlx::item_share(items, grid), per = rlx::part_blocks(cost, lgs, share);
    unsigned long long live = 0, at = 0;
    bool ok = per % (1u << lgs) == 0;
    for (uint32_t part = 0; part < share; ++part) {
      const uint32_t from = part * per;
      if (from >= cost) break;
      ok = ok && from == at;
      at = cost - from < per ? cost : from + per;
      ++live;
    }
    std::printf("%u %llu %d\n", share, live * items, ok && at == cost);
  }
}
