// Host build of the arithmetic and the rule on an image's blocks (csrc/ds_blocks.h, included unchanged).
#include "ds_blocks.h"

extern "C" void blocks_host_place(uint64_t unit, uint32_t units_per_block_log2, uint64_t *out) {
  const DsBlockPlace p = ds_block_place(unit, units_per_block_log2);
  out[0] = p.block;
  out[1] = p.in_block;
}

extern "C" int blocks_host_parts_log2(uint64_t nbytes, uint32_t units_per_block_log2) {
  return ds_block_parts_log2(nbytes, units_per_block_log2);
}
