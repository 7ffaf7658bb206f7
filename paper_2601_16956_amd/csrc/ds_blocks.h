// The blocks that an image is cut into for ds_image_compress: which of them a 16-byte unit lies in, and where in it.
//
// In 64 bits: any power of two of bytes is a block size, so the shift can be by up to 59, for images of any size.  The file
// compiles for the device and, unchanged, for the host, where a test includes it.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define DS_BLOCKS_FN __host__ __device__ __forceinline__
#else
#define DS_BLOCKS_FN static inline
#endif

struct DsBlockPlace {
  uint64_t block, in_block;  // in units
};
DS_BLOCKS_FN DsBlockPlace ds_block_place(uint64_t unit, uint32_t units_per_block_log2) {
  const uint64_t block = unit >> units_per_block_log2;
  return DsBlockPlace{block, unit - (block << units_per_block_log2)};
}
