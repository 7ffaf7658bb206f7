// Host build of the order of a launch's blocks (csrc/ds_perm.h, included unchanged).
#include "ds_perm.h"

// Counts in `hits` how often each of n blocks is taken; returns the work-groups of the launch.
extern "C" uint32_t order_host_deal(uint32_t n, int pack, uint8_t *hits) {
  const DsPermOrder o = ds_perm_order(n, pack != 0);
  for (uint32_t w = 0; w < 8 * o.span; ++w) {
    const uint32_t i = ds_perm_ordered(w, o.stripe, o.magic);
    if (i < n) ++hits[i];
  }
  return 8 * o.span;
}
