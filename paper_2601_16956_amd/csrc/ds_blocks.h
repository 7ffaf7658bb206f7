// The blocks that an image is cut into for ds_image_compress.  The file compiles for the device and, unchanged, for the
// host, where a test includes it.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define DS_BLOCKS_FN __host__ __device__ __forceinline__
#else
#define DS_BLOCKS_FN static inline
#endif

// Which block a 16-byte unit lies in, and where in it.  In 64 bits: any power of two of bytes is a block size, so the shift
// can be by up to 59, for images of any size.
struct DsBlockPlace {
  uint64_t block, in_block;  // in units
};
DS_BLOCKS_FN DsBlockPlace ds_block_place(uint64_t unit, uint32_t units_per_block_log2) {
  const uint64_t block = unit >> units_per_block_log2;
  return DsBlockPlace{block, unit - (block << units_per_block_log2)};
}

// A look for a block that is not constant takes segments of up to 64 KiB ...
constexpr uint32_t kSegmentUnitsLog2 = 12;
// ... or, in images of up to 16 MiB, blocks of 128 KiB to 1 MiB whole, by one work-group or four.  The work-groups per block, as
// a power of two; -1: segments.  (ds_constant_blocks_kernel says why.)
constexpr uint64_t kWholeBlocksBytes = 16ull << 20;
constexpr uint32_t kWholeBlockUnitsLog2 = 16, kOnePartUnitsLog2 = 14, kBlockPartsLog2 = 2;
DS_BLOCKS_FN int ds_block_parts_log2(uint64_t nbytes, uint32_t units_per_block_log2) {
  if (units_per_block_log2 <= kSegmentUnitsLog2 || units_per_block_log2 > kWholeBlockUnitsLog2 || nbytes > kWholeBlocksBytes) return -1;
  return units_per_block_log2 <= kOnePartUnitsLog2 ? 0 : (int)kBlockPartsLog2;
}
