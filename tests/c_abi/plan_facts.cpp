// What a plan holds and which rules its launches follow, read from the library's own plan objects (csrc/ds_internal.h,
// included unchanged) for the tests of those rules.
#include "ds_internal.h"

extern "C" void plan_facts(const ds_plan *p, uint64_t *out) {
  const bool blocks = !p->perms.empty();
  out[0] = p->n_chunks();
  out[1] = p->n_general;
  out[2] = p->n_perm_chunks;
  out[3] = p->perms.size();
  out[4] = p->perm_items.size();
  out[5] = p->rest_recs.size();
  out[6] = p->mostly_general(blocks);
  out[7] = p->scatter_in_pieces(p->n_chunks());
  out[9] = p->n_dims;
  out[10] = p->mostly_several(blocks);
  out[11] = p->mostly_columns();
  out[12] = p->mostly_rests(true);
  out[13] = p->mostly_rests(false);
  out[14] = p->mostly_far();
  out[8] = 0;  // views whose units in the general path are moved an element per lane
  for (const DsTileHot &h : p->hot) out[8] += (h.meta & DS_HOT_LANES) != 0;
}
