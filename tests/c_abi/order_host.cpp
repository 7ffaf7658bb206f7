// Host build of the order of a launch's blocks (csrc/ds_perm.h, included unchanged).
#include "ds_perm.h"

static uint32_t deal(uint32_t n, const DsPermOrder &o, uint8_t *hits) {
  for (uint32_t w = 0; w < 8 * o.span; ++w) {
    const uint32_t i = ds_perm_ordered(w, o.stripe, o.magic);
    if (i < n) ++hits[i];
  }
  return 8 * o.span;
}

// Counts in `hits` how often each of n blocks is taken; returns the work-groups of the launch.
extern "C" uint32_t order_host_deal(uint32_t n, int pack, uint8_t *hits) { return deal(n, ds_perm_order(n, pack != 0), hits); }
extern "C" uint32_t order_host_deal_together(uint32_t n, int pack, uint8_t *hits) {
  return deal(n, ds_perm_order(n, pack != 0, true), hits);
}
// Neighbouring blocks that an XCD takes one after the other.
extern "C" uint32_t order_host_stripe(uint32_t n, int pack, int together) {
  return ds_perm_order(n, pack != 0, together != 0).stripe;
}
