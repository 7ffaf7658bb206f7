// Gather (pack) and scatter (unpack) kernels for gfx950.
//
// The image is cut into chunks of 2^chunk_log2 bytes; one work-group moves one
// chunk (DataStates-LLM Sec. V-A1 coalesces the shards of a checkpoint into
// one region; Sec. V-A4: a chunk need not be a whole tensor).  Work is laid
// out in DESTINATION space: thread -> 16-byte unit of the image, so image
// accesses are aligned, contiguous 16-byte vector accesses whatever the
// shards look like, and every work-group moves the same number of bytes
// however fragmented its part of the image is.
//
// One kernel serves a pack (or unpack) call; a work-group takes (a piece of) one chunk down one of two paths:
// ds_unit_kernel, one unit per thread, in a default call; ds_move_kernel, several units per thread, in plans of
// contiguous shards only, most of whose chunks hold several (they have a simpler second path, multi_chunk), and with
// the options for comparison (other chunk sizes, a grid limit, the variants).  Views with runs shorter than 16 bytes
// are moved by a kernel of their own, ds_perm_kernel.
//
// lean path: a thread issues all its loads, then all its stores, and is done.  Many short-lived work-groups keep the
//   addresses in flight inside a compact, moving window of HBM: measured on MI355X a plain copy of one unit per thread
//   and eight wavefronts per SIMD runs at 6.75 TB/s (read+write), of four units and four wavefronts at 6.3, and one
//   whose work-groups stream through 64-256 KiB each at 5.3.  Everything the path
//   needs for a chunk is one 32-byte record prepared by the plan (DsChunkRec),
//   so the only dependent load before the data is that record.  It handles the
//   chunks that are whole units of one tile (contiguous, or rows of a 2-D view
//   of at least 16 bytes each).
//
// general path: the remaining chunks (tile boundaries, payload tails, padding,
//   N-D views); their record names the tiles they hold.  The tiles are taken
//   64 at a time: the first wavefront reads one tile's compact descriptor
//   (DsTileHot, 40 bytes) per lane, a wavefront inclusive scan over the unit
//   counts turns the 64 tiles into one dense index space, and the threads of
//   the work-group share that space evenly, one unit each per pass (ds_move_kernel: up to four), in three
//   phases: (1) registers and LDS only: find the tile of each unit by binary
//   search over the scan and classify it; (2) all loads, nothing between
//   them; (3) all stores.  Chunks inside a view with several outer dimensions
//   and runs of 16 bytes and more need none of that: ds_unit_kernel moves them
//   by their record (dims_move); ds_move_kernel takes large pieces of such views
//   out of the scan and walks them with the whole work-group ("direct").
//
// Tensor-side addresses are only element-aligned.  gfx950 runs with unaligned
// global access enabled, so a 16-byte unit that lies inside one contiguous run
// is one (possibly unaligned) dwordx4 access; a unit that is cut by the end of
// a run or of the payload is assembled from 16-byte loads that lie inside the
// runs (gather), stored in pieces that cover exactly its bytes (scatter), or,
// for runs shorter than 16 bytes, moved piece by piece, so no byte outside
// the described views is ever read or written.

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "ds_internal.h"
#include "ds_blocks.h"
#include "ds_splice.h"

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_unaligned __attribute__((aligned(1)));

constexpr int kWave = 64;
// Beside a launch of blocks (ds_perm_kernel): the launch of the other chunks takes a list of them, or passes over the
// few chunks the blocks cover.
enum : int { kAlone = 0, kBeside = 1, kListed = 2 };
constexpr uint32_t kUnitPieces = 4;       // work-groups of ds_unit_kernel per chunk
// Images of at most so many bytes are moved with ordinary loads, larger ones with non-temporal ones, which leave nothing
// in the 256 MB last-level cache.  Copies of one unit per thread, three pairs of buffers in turn, ordinary / non-
// temporal: 23 MB 7.4 / 8.4 us, 40 MB 11.9 / 14.5, 58 MB 16.6 / 20.6, 70 MB 19.7 / 23.2, 85 MB 27.1 / 27.7, 110 MB (nothing
// is found again) 36.8 / 34.6, 1.5 GB 476 / 453.  What that gains is the second pass over the same bytes: it is a property of
// that rotation as much as of the cache.  On bytes that no cache holds (the gather and the scatter over tables, images
// and tensors of 700 MB in rotation) ordinary loads cost 3 to 26 %: one tensor of 5 MB 4.05 / 3.78 and 3.80 / 3.02, of 23 MB
// 11.6 / 10.5 and 11.4 / 9.8, of 60 MB 24.1 / 22.0 and 24.3 / 22.0, a 27 MB training state 12.8 / 11.6 and 12.2 / 10.7; and a
// plain copy behind a pass that reads and writes its source 5 MB 3.1 / 3.1, 23 MB 12.7 / 10.5, 40 MB 11.4 / 15.5, 60 MB 17.6 / 20.7.
constexpr uint64_t kCachedBytes = 64ull << 20;
constexpr uint32_t kBigUnits = 512;       // N-D views: pieces of >= 8 KiB inside a chunk leave the scan

// A kernel's arguments up to its first structure are in scalar registers when a wavefront starts (build.py asks for it, up to
// 14 registers); the others it reads itself.  So what leads to a work-group's record or block comes first and by itself,
// and what only some work-groups need is in structures.  Read / in registers, us: scatter of 23 MB in 106 tensors 8.8 / 8.3,
// gather 8.6 / 8.5; 7.5 GB in 20 000 fragments 2316 / 2310; 8000 squares of 24 bf16 23.9 / 23.4 and 26.2 / 25.5; views of 592
// columns of 8 bytes 7.4 / 7.1.
struct MoveArgs {
  const DsTile *tiles;
  const DsTileHot *hot;  // n_tiles + 1 entries: the general path's compact copy of the tiles, and a sentinel
  const uint32_t *first_tile;
  uint8_t *img;         // points at image byte img_lo
  uint64_t img_lo, img_hi;
  uint64_t total;       // image length
  uint32_t chunk_log2;
  uint32_t n_extra;     // 0..2 chunks cut by img_lo / img_hi: they take the general path whatever their kind
                        // (pieces of chunks: | log2(pieces per chunk) << 8).  Both
                        // structures together have 120 bytes: with 128 the 23 MB gather took 0.2 us longer
  uint32_t extra[2];
};

struct LeanArgs {
  const DsChunkRec *recs;
  const uint32_t *ids; // kListed launches: the chunk a record belongs to
  uint8_t *img;        // points at image byte img_lo
  uint64_t img_lo;
  uint32_t chunk_log2;
  uint32_t c_lo;       // record of the first whole chunk inside [img_lo, img_hi)
  uint32_t n_pieces;   // work-groups' pieces of the whole chunks inside the range
  uint32_t xcd_span;   // pieces per XCD (ceil(n_pieces / 8)); 0 = work-group i takes piece i
};

// ---- 16-byte accesses -------------------------------------------------------
// Every address here is device (or pinned host) memory reached through the global address space; saying so
// makes the compiler emit global_load / global_store instead of the flat forms, which also have to ask
// whether the address lies in LDS or scratch.
#define DS_GLOBAL __attribute__((address_space(1)))
template <bool NT>
__device__ __forceinline__ u32x4 ld16_aligned(const uint8_t *p) {
  if (NT) return __builtin_nontemporal_load((const DS_GLOBAL u32x4 *)p);
  return *(const DS_GLOBAL u32x4 *)p;
}
template <bool NT>
__device__ __forceinline__ void st16_aligned(uint8_t *p, u32x4 v) {
  if (NT) __builtin_nontemporal_store(v, (DS_GLOBAL u32x4 *)p);
  else *(DS_GLOBAL u32x4 *)p = v;
}
template <bool NT>
__device__ __forceinline__ u32x4 ld16_any(const uint8_t *p) {
  if (NT) return __builtin_nontemporal_load((const DS_GLOBAL u32x4_unaligned *)p);
  return *(const DS_GLOBAL u32x4_unaligned *)p;
}
template <bool NT>
__device__ __forceinline__ void st16_any(uint8_t *p, u32x4 v) {
  if (NT) __builtin_nontemporal_store(v, (DS_GLOBAL u32x4_unaligned *)p);
  else *(DS_GLOBAL u32x4_unaligned *)p = v;
}

// ---- index arithmetic -------------------------------------------------------
__device__ __forceinline__ void divmod(uint64_t a, uint64_t b, uint64_t &q, uint64_t &r) {
  if (((a | b) >> 32) == 0) {
    uint32_t qq = (uint32_t)a / (uint32_t)b;
    q = qq;
    r = (uint32_t)a - qq * (uint32_t)b;
  } else {
    q = a / b;
    r = a - q * b;
  }
}

// address of the first byte of run number `row` (runs counted in row-major
// order of the outer dimensions)
__device__ __forceinline__ uint64_t run_address(const DsTile *t, uint64_t row) {
  const uint32_t m = t->n_outer;
  if (m == 0) return t->src;
  if (m == 1) return t->src + row * t->stride[0];
  uint64_t a = t->src;
  for (int j = (int)m - 1; j > 0; --j) {
    uint64_t q, r;
    divmod(row, t->extent[j], q, r);
    a += r * t->stride[j];
    row = q;
  }
  return a + row * t->stride[0];
}

// Inclusive scan over the wavefront, by data-parallel moves: inside each row of 16 lanes, then the last lane of rows 0 and
// 2 to the row behind, then that of the first half to the second.  (Through LDS, by __shfl_up, the lanes read from stay in
// registers across the loops around it: 66 in the gather beside blocks, which is launched for eight wavefronts per SIMD.)
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x) {
  const auto add = [&](auto ctrl, auto rows) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, decltype(rows)::value, 0xF, false);
  };
  constexpr std::integral_constant<int, 0xF> all;
  add(std::integral_constant<int, 0x111>(), all);  // row_shr 1, 2, 4, 8
  add(std::integral_constant<int, 0x112>(), all);
  add(std::integral_constant<int, 0x114>(), all);
  add(std::integral_constant<int, 0x118>(), all);
  add(std::integral_constant<int, 0x142>(), std::integral_constant<int, 0xA>());  // row_bcast 15
  add(std::integral_constant<int, 0x143>(), std::integral_constant<int, 0xC>());  // row_bcast 31
  return x;
}

// ---- units cut by the end of a run ------------------------------------------------------
// bytes [s, s+16) of the 32 bytes a||b, 0 < s < 16 (word selects and byte-aligns, see ds_splice.h)
__device__ __forceinline__ u32x4 splice(u32x4 a, u32x4 b, uint32_t s) {
  const DsWords4 r = ds_splice_words(DsWords4{{a.x, a.y, a.z, a.w}}, DsWords4{{b.x, b.y, b.z, b.w}}, s);
  return u32x4{r.w[0], r.w[1], r.w[2], r.w[3]};
}

// The value lane + 1 of the wavefront holds (the last lane keeps its own): one data-parallel move, "wavefront
// shift left by one".
__device__ __forceinline__ uint32_t lane_above(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x130, 0xF, 0xF, false);
}

// the low n < 16 bytes of v to p (any alignment), as one store each of 8, 4, 2 and 1 bytes as n has those bits
typedef uint64_t u64_unaligned __attribute__((aligned(1)));
typedef uint32_t u32_unaligned __attribute__((aligned(1)));
typedef uint16_t u16_unaligned __attribute__((aligned(1)));
__device__ __forceinline__ void store_low_bytes(uint8_t *p, u32x4 v, uint32_t n) {
  uint64_t lo = v.x | ((uint64_t)v.y << 32);
  const uint64_t hi = v.z | ((uint64_t)v.w << 32);
  if (n & 8) {
    *(DS_GLOBAL u64_unaligned *)p = lo;
    p += 8;
    lo = hi;
  }
  if (n & 4) {
    *(DS_GLOBAL u32_unaligned *)p = (uint32_t)lo;
    p += 4;
    lo >>= 32;
  }
  if (n & 2) {
    *(DS_GLOBAL u16_unaligned *)p = (uint16_t)lo;
    p += 2;
    lo >>= 16;
  }
  if (n & 1) *(DS_GLOBAL uint8_t *)p = (uint8_t)lo;
}
// ... and the n < 16 bytes at p, as one load each of 8, 4, 2 and 1 bytes, zeros behind them
__device__ __forceinline__ u32x4 load_low_bytes(const uint8_t *p, uint32_t n) {
  uint32_t f0 = 0, f1 = 0, x = 0, y = 0;
  if (n & 8) {
    const uint64_t first = *(const DS_GLOBAL u64_unaligned *)p;
    f0 = (uint32_t)first;
    f1 = (uint32_t)(first >> 32);
  }
  if (n & 4) x = *(const DS_GLOBAL u32_unaligned *)(p + (n & 8));
  if (n & 2) y = *(const DS_GLOBAL u16_unaligned *)(p + (n & 12));
  if (n & 1) {
    const uint32_t last = *(const DS_GLOBAL uint8_t *)(p + (n & 14));
    y |= n & 2 ? last << 16 : last;
  }
  if (!(n & 4)) {
    x = y;
    y = 0;
  }
  return n & 8 ? u32x4{f0, f1, x, y} : u32x4{x, y, 0, 0};
}
// bytes [0,k) of v go to p0, bytes [k,valid) to p1 (0 < k < 16, k <= valid <= 16); exactly those bytes are written
__device__ __forceinline__ void store_cut(uint8_t *p0, uint8_t *p1, uint32_t k, u32x4 v, uint32_t valid = 16) {
  store_low_bytes(p0, v, k);
  if (valid > k) store_low_bytes(p1, splice(v, u32x4{0, 0, 0, 0}, k), valid - k);
}

// A unit of a view with outer dimensions that lies in several runs, piece by piece: its first `valid` bytes, of which
// the first k (all that is left of run `row`, or 16) are at p.  PACK: tensor -> the unit (its rest stays 0), else the
// unit v -> tensor.  A loop over pieces and not over elements in registers: that took 86 registers and kept every
// kernel with this routine below six wavefronts per SIMD.
template <bool PACK>
__device__ __forceinline__ u32x4 move_runs(const DsTile *t, uint64_t row, uint8_t *p, uint32_t k, uint32_t valid, u32x4 v) {
  const uint32_t run = t->run_bytes < 16 ? (uint32_t)t->run_bytes : 16u;
  uint32_t at = 0;
#pragma unroll 1
  while (true) {
    const uint32_t n = k < valid - at ? k : valid - at;
    if (PACK) {
      const u32x4 x = load_low_bytes(p, n);
      v |= at ? splice(u32x4{0, 0, 0, 0}, x, 16u - at) : x;
    } else {
      store_low_bytes(p, at ? splice(v, u32x4{0, 0, 0, 0}, at) : v, n);
    }
    at += n;
    if (at >= valid) return v;
    p = reinterpret_cast<uint8_t *>(run_address(t, ++row));
    k = run;
  }
}

// ---- one unit, any tile, any position (the general routine) ------------------
// x: image offset of the unit (multiple of 16) inside tile t's range; imgp: its
// address in the image buffer.
template <bool PACK, bool NTL, bool NTS>
__device__ __forceinline__ void move_unit(const DsTile *t, uint64_t tile_begin, uint64_t x, uint8_t *imgp) {
  const uint64_t nbytes = t->nbytes;
  const uint64_t b = x - tile_begin;
  if (b >= nbytes) {  // padding
    if (PACK) st16_aligned<NTS>(imgp, u32x4{0, 0, 0, 0});
    return;
  }
  const uint64_t left = nbytes - b;
  const uint32_t valid = left < 16 ? (uint32_t)left : 16u;
  const uint64_t L = t->run_bytes;
  uint64_t row = 0, col = b;
  if (t->n_outer) divmod(b, L, row, col);
  uint8_t *const p = reinterpret_cast<uint8_t *>(run_address(t, row) + col);
  if (valid == 16 && col + 16 <= L) {
    if (PACK) st16_aligned<NTS>(imgp, ld16_any<NTL>(p));
    else st16_any<NTS>(p, ld16_aligned<NTL>(imgp));
    return;
  }
  const uint32_t k = L - col < 16 ? (uint32_t)(L - col) : 16u;
  if (PACK) st16_aligned<NTS>(imgp, move_runs<true>(t, row, p, k, valid, u32x4{0, 0, 0, 0}));
  else (void)move_runs<false>(t, row, p, k, valid, ld16_aligned<NTL>(imgp));
}

// ---- units of views with runs shorter than 16 bytes, an element per lane ----------------------------------
// For DS_HOT_LANES: the few units that such views leave to the general path while everything else is under way.  Bound by
// latency: move_unit has one piece of a unit after the other, up to 16, each behind the tile's descriptor again, and a
// launch that holds one such unit ends with it.  Here the elements of a wavefront's units are dealt to its lanes, and the
// descriptor is read once.  Piece by piece / by lanes, us: a state of 20 MB with one view of 400 transposed bytes, gather
// 23.5 / 15.4, scatter 23.2 / 15.0; of 40 MB with a transposed matrix of 2 KB 24.7 / 21.6 and 23.7 / 23.3.
// `units`: a mask of the wavefront's lanes that hold one, of tile bt + q, `off` bytes behind cb in the image, which is at
// cimg.  They are taken tile by tile, so that the descriptor is in scalar registers.
#define DS_CONSTANT __attribute__((address_space(4)))
template <typename E, bool PACK>
__device__ __forceinline__ void move_elements_by_lanes(const DS_CONSTANT DsTile *t, uint32_t before_cb, uint8_t *cimg,
                                                       uint32_t lane, uint32_t n, uint32_t list) {
  constexpr uint32_t kPerUnit = 16 / sizeof(E), kStep = kWave / kPerUnit;
  constexpr int kAhead = PACK ? 2 : 3;  // loads a lane has under way: more take registers that six wavefronts of ds_move_kernel do not have
  const uint32_t in_unit = lane % kPerUnit * (uint32_t)sizeof(E), run = (uint32_t)t->run_bytes;
#pragma unroll 1
  for (uint32_t base = 0; base < n; base += kAhead * kStep) {
    uint64_t p[kAhead];   // the element's address; 0: padding, or no unit
    uint32_t at[kAhead];  // its place in the image, from cimg; ~0: no unit
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      const uint32_t k = base + i * kStep + lane / kPerUnit;
      const uint32_t unit = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(k * 4), (int)list);  // (of lane k mod 64)
      p[i] = 0;
      at[i] = ~0u;
      if (k < n) {
        at[i] = unit + in_unit;
        const uint32_t b = before_cb + at[i];
        if (b < (uint32_t)t->nbytes) {
          uint32_t row = b / run;
          uint64_t x = t->src + (b - row * run);
#pragma unroll 1
          for (uint32_t j = t->n_outer - 1; j > 0; --j) {
            const uint32_t extent = (uint32_t)t->extent[j], rows = row / extent;
            x += (row - rows * extent) * t->stride[j];
            row = rows;
          }
          p[i] = x + row * t->stride[0];
        }
      }
    }
    E v[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      v[i] = 0;
      if (p[i]) v[i] = PACK ? *(const DS_GLOBAL E *)p[i] : *(const DS_GLOBAL E *)(cimg + at[i]);
    }
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      if (PACK && at[i] != ~0u) *(DS_GLOBAL E *)(cimg + at[i]) = v[i];
      if (!PACK && p[i]) *(DS_GLOBAL E *)p[i] = v[i];
    }
  }
}
template <bool PACK>
__device__ __forceinline__ void move_by_lanes(const MoveArgs &a, uint32_t bt, uint64_t cb, uint8_t *cimg, uint64_t units,
                                              uint32_t q, uint32_t off) {
  uint32_t lane = threadIdx.x & (kWave - 1);
  asm volatile("" : "+v"(lane));  // nothing made of it is kept in registers while the other units are moved
#pragma unroll 1
  while (units) {
    const uint32_t q0 = (uint32_t)__builtin_amdgcn_readlane((int)q, __builtin_ctzll(units));
    const uint64_t here = units & __ballot(q == q0);
    units &= ~here;
    const uint32_t n = (uint32_t)__builtin_popcountll(here);
    // lane r gets the r-th unit: its owner sends it there, and the others send to the lanes behind
    const uint32_t before = __builtin_amdgcn_mbcnt_hi((uint32_t)(here >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)here, 0));
    const uint32_t to = here >> lane & 1 ? before : n + lane - before;
    const uint32_t list = (uint32_t)__builtin_amdgcn_ds_permute((int)(to * 4), (int)off);
    const DS_CONSTANT DsTile *t = (const DS_CONSTANT DsTile *)(uintptr_t)(a.tiles + bt) + q0;
    // (a view of less than 4 GiB: 32 bits hold the distance modulo 2^32, and what it is added to brings it into the view)
    const uint32_t before_cb = (uint32_t)(cb - ((const DS_CONSTANT DsTileHot *)(uintptr_t)(a.hot + bt) + q0)->img_off);
    switch (t->es_log2) {
      case 0: move_elements_by_lanes<uint8_t, PACK>(t, before_cb, cimg, lane, n, list); break;
      case 1: move_elements_by_lanes<uint16_t, PACK>(t, before_cb, cimg, lane, n, list); break;
      case 2: move_elements_by_lanes<uint32_t, PACK>(t, before_cb, cimg, lane, n, list); break;
      default: move_elements_by_lanes<uint64_t, PACK>(t, before_cb, cimg, lane, n, list); break;
    }
  }
}

// ---- direct path: one tile range, whole work-group ---------------------------
// [lo, hi): image range of the tile clipped to the chunk, multiples of 16.
template <bool PACK, int NT, int UNROLL, bool NTL, bool NTS>
__device__ __forceinline__ void move_tile_direct(const DsTile *t, uint64_t tile_begin, uint64_t lo, uint64_t hi,
                                                 uint8_t *img, uint64_t img_lo) {
  const uint32_t tid = threadIdx.x;
  const uint64_t nbytes = t->nbytes;
  const uint64_t full_end = tile_begin + (nbytes & ~(uint64_t)15);  // image offset where whole payload units end
  const uint32_t n_all = (uint32_t)((hi - lo) >> 4);
  uint32_t n_full = 0;
  if (full_end > lo) n_full = (uint32_t)(((full_end < hi ? full_end : hi) - lo) >> 4);
  uint8_t *imgp = img + (lo - img_lo);
  const uint64_t b0 = lo - tile_begin;
  const uint32_t m = t->n_outer;

  if (m == 0) {
    uint8_t *s = reinterpret_cast<uint8_t *>(t->src + b0);
    for (uint32_t base = 0; base < n_full; base += NT * UNROLL) {
      u32x4 v[UNROLL];
#pragma unroll
      for (int i = 0; i < UNROLL; ++i) {
        const uint32_t u = base + i * NT + tid;
        if (u < n_full) v[i] = PACK ? ld16_any<NTL>(s + 16ull * u) : ld16_aligned<NTL>(imgp + 16ull * u);
      }
#pragma unroll
      for (int i = 0; i < UNROLL; ++i) {
        const uint32_t u = base + i * NT + tid;
        if (u < n_full) {
          if (PACK) st16_aligned<NTS>(imgp + 16ull * u, v[i]);
          else st16_any<NTS>(s + 16ull * u, v[i]);
        }
      }
    }
  } else {
    const uint64_t L = t->run_bytes;
    uint64_t row0, col0;
    divmod(b0, L, row0, col0);
    if (L < (1ull << 31)) {
      const uint32_t L32 = (uint32_t)L, c32 = (uint32_t)col0;
      for (uint32_t base = 0; base < n_full; base += NT * UNROLL) {
#pragma unroll
        for (int i = 0; i < UNROLL; ++i) {
          const uint32_t u = base + i * NT + tid;
          if (u < n_full) {
            const uint32_t tt = c32 + 16u * u;        // < 2^31 + 2^22
            const uint32_t q = tt / L32;
            const uint32_t col = tt - q * L32;
            const uint64_t row = row0 + q;
            uint8_t *ip = imgp + 16ull * u;
            uint8_t *const p = reinterpret_cast<uint8_t *>(run_address(t, row) + col);
            if (col + 16u <= L32) {
              if (PACK) st16_aligned<NTS>(ip, ld16_any<NTL>(p));
              else st16_any<NTS>(p, ld16_aligned<NTL>(ip));
            } else {
              if (PACK) st16_aligned<NTS>(ip, move_runs<true>(t, row, p, L32 - col, 16, u32x4{0, 0, 0, 0}));
              else (void)move_runs<false>(t, row, p, L32 - col, 16, ld16_aligned<NTL>(ip));
            }
          }
        }
      }
    } else {
      for (uint32_t u = tid; u < n_full; u += NT)
        move_unit<PACK, NTL, NTS>(t, tile_begin, lo + 16ull * u, imgp + 16ull * u);
    }
  }
  // the unit cut by the end of the payload, then padding
  for (uint32_t u = n_full + tid; u < n_all; u += NT)
    move_unit<PACK, NTL, NTS>(t, tile_begin, lo + 16ull * u, imgp + 16ull * u);
}

// Image bytes [cb, ce) of chunk c (WHOLE), or of its piece of BYTES from byte `piece` on, that lie in the launch's range;
// false if none do.
template <bool WHOLE, uint32_t BYTES>
__device__ __forceinline__ bool piece_range(const MoveArgs &a, uint64_t c, uint32_t piece, uint64_t &cb, uint64_t &ce) {
  const uint64_t c_begin = (c << a.chunk_log2) + (WHOLE ? 0u : piece);
  uint64_t c_end = WHOLE ? (c + 1) << a.chunk_log2 : c_begin + BYTES;
  if (c_end > a.total) c_end = a.total;
  cb = c_begin > a.img_lo ? c_begin : a.img_lo;
  ce = c_end < a.img_hi ? c_end : a.img_hi;
  return cb < ce;
}

// What a batch of up to 64 tiles of a general chunk needs, staged in LDS by the first wavefront.  Everything
// a unit needs is relative to the start of its tile's range inside the (clipped) chunk, so that the per-unit
// arithmetic is 32-bit: a chunk is at most 32 KiB.
struct GenLds {
  uint32_t incl[kWave];   // inclusive scan of the tiles' unit counts inside the chunk
  uint32_t begin[kWave];  // where a tile's clipped range starts, relative to the chunk's clipped start
  uint32_t rem[kWave];    // payload bytes from there on (clamped to 2^31; 0 = padding only)
  uint32_t run[kWave];    // views with one outer dimension: run length
  uint32_t col0[kWave];   // ... and the position of the clipped start inside its run
  uint32_t meta[kWave];   // n_outer | log2(itemsize) << 8 | kRunGe16 if the runs are at least 16 bytes long | DS_HOT_*
  uint64_t src0[kWave];   // address of the clipped start (one run), or of the start of the run that holds it
  uint64_t pitch[kWave];  // views with one outer dimension: distance between runs
  uint64_t big_mask;      // tiles taken out of the scan (large pieces of views with several outer dimensions)
  uint32_t n_units;       // units of the batch = incl[63]
};
constexpr uint32_t kRunGe16 = 1u << 16;
constexpr int kStorePolicySc0Sc1Nt = 1 | 2 | 16;  // sc0 | nt | sc1 in the buffer-store intrinsic's aux operand
// s_waitcnt immediate on gfx9: vmcnt = 0 (bits 3:0 and 15:14), expcnt (6:4) and lgkmcnt (11:8) left at their maxima
constexpr int kWaitVmcnt0 = 0x0F70;

// One general chunk, whole work-group: chunk number c, which holds (parts of) tiles t0 .. t1.
//
// The tiles are taken 64 at a time.  The first wavefront reads their compact descriptors (DsTileHot, one tile
// per lane), turns the unit counts into one dense index space with an inclusive scan, and leaves what the
// units need in LDS; then every thread takes the units tid, tid + NT, ... of that space, UNROLL at a time in
// phases: find the tile of each unit (binary search over the scan) and classify it, issue all loads, issue
// all stores.  So a chunk costs three dependent trips to memory (record -> descriptors -> data) however many
// tiles it holds.  Units that are one 16-byte access (inside the payload of a contiguous tile or inside a row
// of a 2-D view), padding, and units cut by the end of a run of at least 16 bytes are handled in the phases;
// only the rest (runs shorter than 16 bytes, views with several outer dimensions) goes afterwards, an element per lane
// where the plan has little of it (DS_HOT_LANES), else one by one through
// move_unit.
// BLOCKS (not kAlone): a launch of blocks moves the views marked DS_HOT_PERM.
template <bool PACK, int NT, int UNROLL, bool NTL, bool NTS, bool BUFST, int BLOCKS, bool WHOLE>
__device__ __forceinline__ void general_chunk(const MoveArgs &a, uint64_t c, uint32_t piece, uint32_t t0, uint32_t t1,
                                              GenLds *g) {
  const uint32_t tid = threadIdx.x;
  const uint32_t lane = tid & (kWave - 1);
  uint64_t cb, ce;
  if (!piece_range<WHOLE, NT * UNROLL * 16>(a, c, piece, cb, ce)) return;
  uint8_t *const cimg = a.img + (cb - a.img_lo);  // the chunk's (clipped) start in the image buffer
  // Gather with buffer stores: the resource covers exactly the chunk's part of the image, and a lane that has
  // nothing to store in a phase gives an offset beyond it, which the hardware drops.  The stores of a phase
  // are then plain instructions one behind the other, with no branch (and no wait) between them.
  __amdgpu_buffer_rsrc_t image_rsrc;
  if (PACK && BUFST) image_rsrc = __builtin_amdgcn_make_buffer_rsrc(cimg, 0, (int)(uint32_t)(ce - cb), 0x00020000);
  constexpr uint32_t kNoStore = 0x80000000u;

  for (uint32_t bt = t0; bt <= t1; bt += kWave) {
    __syncthreads();  // readers of the previous batch (or of the previous chunk) are done
    if (tid < kWave) {
      const uint32_t ti = bt + lane;
      uint64_t lo = cb, hi = cb, tb = cb;
      uint64_t src = 0, nbytes = 0, stride0 = 0;
      uint32_t run = 0, meta = 0;
      if (ti <= t1) {
        const DsTileHot *h = a.hot + ti;
        tb = h->img_off;
        src = h->src;
        nbytes = h->nbytes;
        stride0 = h->stride0;
        run = h->run;
        meta = h->meta;
        const uint64_t te = h[1].img_off;  // the entry behind the last tile is a sentinel
        lo = tb > cb ? tb : cb;
        if (BLOCKS && (meta & DS_HOT_PERM)) {  // its whole units are moved in blocks: the cut unit and padding are left
          const uint64_t rest = tb + (nbytes & ~(uint64_t)15);
          lo = rest > lo ? rest : lo;
        }
        hi = te < ce ? te : ce;
        if (hi < lo) hi = lo;
      }
      const uint32_t n_outer = meta & 0xFFu;
      const uint32_t units = (uint32_t)((hi - lo) >> 4);
      // (of a view that is moved in blocks only padding can be large: that is what the scan's units write fastest)
      const bool big = UNROLL > 1 && NT * UNROLL >= kBigUnits && units >= kBigUnits && n_outer > 1 && !(BLOCKS && (meta & DS_HOT_PERM));
      const uint64_t big_mask = __ballot(big);
      const uint32_t incl = wave_inclusive_scan(big ? 0u : units);
      const uint64_t b0 = lo - tb;  // byte of the tile's own range at which its clipped range starts
      uint64_t rem = b0 < nbytes ? nbytes - b0 : 0;
      if (rem > (1ull << 31)) rem = 1ull << 31;
      uint64_t src0 = src + b0;
      uint32_t col0 = 0;
      uint64_t longest = nbytes;  // length of the tile's runs
      if (n_outer == 1) {
        uint64_t row0, c0;
        divmod(b0, run, row0, c0);
        src0 = src + row0 * stride0;
        col0 = (uint32_t)c0;
        longest = run;
      }
      g->incl[lane] = incl;
      g->begin[lane] = (uint32_t)(lo - cb);
      g->rem[lane] = (uint32_t)rem;
      g->run[lane] = run;
      g->col0[lane] = col0;
      g->meta[lane] = meta | (longest >= 16 ? kRunGe16 : 0u);
      g->src0[lane] = src0;
      g->pitch[lane] = stride0;
      if (lane == kWave - 1) {
        g->n_units = incl;
        g->big_mask = big_mask;
      }
    }
    __syncthreads();
    const uint32_t n_units = g->n_units;
    for (uint32_t base = 0; base < n_units; base += NT * UNROLL) {
      // how[i]: kind | k << 8 | last << 16 | tile << 24 (k: bytes of a cut unit that end its run; last: the
      // payload ends with that run; tile: 0..63 inside the batch)
      enum : uint32_t { kNone = 0, kFast = 1, kZero = 2, kCut = 3, kSlow = 4, kCutHeld = 5, kTiny = 6, kKind = 0xFFu, kLast = 1u << 16 };
      uint32_t j[UNROLL], p[UNROLL], how[UNROLL];
      uint8_t *ip[UNROLL];   // the unit in the image buffer
      uint8_t *sp[UNROLL];   // kFast, kCut: where the unit starts in the tensor
      // ---- phase 1, registers and LDS only: which tile each unit belongs to, and what kind of unit it is ----
      // A thread's i-th unit of the pass.  Each block of NT units is rotated by 9 more than the one before:
      // tensors of one size put their cut units at a fixed period, and periods that divide NT (slots of 512
      // bytes to 4 KiB) would otherwise give all of them to the same few threads, four each.
#pragma unroll
      for (int i = 0; i < UNROLL; ++i) {
        j[i] = base + i * NT + ((tid + 40u * i) & (NT - 1));
        p[i] = 0;
      }
      // smallest p with incl[p] > j, the searches of the thread's units side by side (a unit beyond the end
      // of the batch ends at tile 63: every index stays inside the table)
#pragma unroll
      for (int step = kWave / 2; step > 0; step >>= 1) {
#pragma unroll
        for (int i = 0; i < UNROLL; ++i)
          if (g->incl[p[i] + step - 1] <= j[i]) p[i] += step;
      }
#pragma unroll
      for (int i = 0; i < UNROLL; ++i) {
        how[i] = kNone;
        ip[i] = cimg;
        sp[i] = cimg;
        if (j[i] < n_units) {
          const uint32_t q = p[i];
          const uint32_t d = 16u * (j[i] - (q ? g->incl[q - 1] : 0u));  // the unit's offset in the tile's clipped range
          ip[i] = cimg + (g->begin[q] + d);
          const uint32_t rem = g->rem[q];
          const uint32_t meta = g->meta[q];
          if (d >= rem) {
            how[i] = kZero;
          } else if ((meta & 0xFFu) > 1 || !(meta & kRunGe16)) {
            how[i] = kSlow | (q << 24);
            if (!(meta & 0xFFu)) {
              how[i] = kTiny | (rem << 8);
              sp[i] = reinterpret_cast<uint8_t *>(g->src0[q]);
            }
          } else {
            // the run the unit starts in: what is left of the payload, or one row of a 2-D view
            uint64_t run0 = g->src0[q];
            uint32_t L = rem, col = d;
            if (meta & 0xFFu) {
              L = g->run[q];
              const uint32_t t = g->col0[q] + d;  // < 2^31 + 2^15
              const uint32_t rows = t / L;
              col = t - rows * L;
              run0 += (uint64_t)rows * g->pitch[q];
            }
            sp[i] = reinterpret_cast<uint8_t *>(run0 + col);
            if (col + 16u <= L) {
              how[i] = kFast;
            } else {
              const uint32_t k = L - col;
              // unless the payload ends with this run, the unit goes on in the next one
              const bool last = !(meta & 0xFFu) || d + k >= rem;
              how[i] = kCut | (k << 8) | (last ? kLast : 0u) | (q << 24);
            }
          }
        }
      }
      // Gather: the thread's first cut unit of the pass travels with the others: its two loads are issued in
      // the load phase, it is spliced into v[] and leaves with the same store instruction as its neighbours
      // (so that a line of the image is written whole).  Further cut units of the same thread wait for a
      // phase of their own; the rotation above makes them rare.  (Chosen here, after the units have been
      // classified independently of each other, so that their classifications can run side by side.)
      bool cut_held = false;
      uint8_t *cut_pa = nullptr, *cut_pb = nullptr;  // the last 16 bytes of the run; the first 16 of the next (or null)
      if (PACK) {
#pragma unroll
        for (int i = 0; i < UNROLL; ++i)
          if ((how[i] & kKind) == kCut && !cut_held) {
            cut_held = true;
            const uint32_t k = (how[i] >> 8) & 0xFFu, q = how[i] >> 24;
            cut_pa = sp[i] + k - 16;
            if (!(how[i] & kLast)) cut_pb = sp[i] + k + (g->pitch[q] - g->run[q]);
            how[i] = kCutHeld | (k << 8);
          }
      }
      // ---- phase 2: all loads, nothing between them ----
      u32x4 v[UNROLL];
#pragma unroll
      for (int i = 0; i < UNROLL; ++i) v[i] = u32x4{0, 0, 0, 0};  // padding is written as zeros
      u32x4 cut_a = u32x4{0, 0, 0, 0}, cut_b = u32x4{0, 0, 0, 0};
#pragma unroll
      for (int i = 0; i < UNROLL; ++i) {
        const uint32_t kind = how[i] & kKind;
        if (PACK) {
          if (kind == kFast) v[i] = ld16_any<NTL>(sp[i]);
          if (UNROLL == 1 && kind == kTiny) v[i] = load_low_bytes(sp[i], how[i] >> 8);
        } else {
          if (kind == kFast || kind == kCut || kind == kTiny) v[i] = ld16_aligned<NTL>(ip[i]);
        }
      }
      if (PACK && cut_held) {
        cut_a = ld16_any<NTL>(cut_pa);
        if (cut_pb) cut_b = ld16_any<NTL>(cut_pb);
      }
      // ---- phase 3: all stores ----
      // Every load has landed before the first store goes out.  Loads and stores share one counter and
      // complete out of order with respect to each other, so a wait for a load that is issued behind a store
      // waits for that store as well; left to itself the compiler, which cannot tell on every path that the
      // loads are done, puts such a wait in front of each store and the stores leave one round trip apart.
      __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
      if (PACK && UNROLL > 1) {
        // Tensors of less than 16 bytes, read once the other loads have landed: a lane's v[i] would have to wait for the
        // load that is under way for its neighbours' (60 000 tensors of 128 bytes beside a view, of which none is that
        // small: 7.4 us with these loads among the others, as it is 7.2; in chunks of 32 KiB 12.0 and 11.5)
        bool tiny = false;
#pragma unroll
        for (int i = 0; i < UNROLL; ++i) tiny |= (how[i] & kKind) == kTiny;
        if (__ballot(tiny)) {
#pragma unroll
          for (int i = 0; i < UNROLL; ++i)
            if ((how[i] & kKind) == kTiny) v[i] = load_low_bytes(sp[i], how[i] >> 8);
        }
      }
      if (PACK) {
        if (cut_held) {
          uint32_t k = 0;
#pragma unroll
          for (int i = 0; i < UNROLL; ++i)
            if ((how[i] & kKind) == kCutHeld) k = (how[i] >> 8) & 0xFFu;
          const u32x4 spliced = splice(cut_a, cut_b, 16u - k);
#pragma unroll
          for (int i = 0; i < UNROLL; ++i)
            if ((how[i] & kKind) == kCutHeld) v[i] = spliced;
        }
#pragma unroll
        for (int i = 0; i < UNROLL; ++i) {
          const uint32_t kind = how[i] & kKind;
          const bool stores = kind == kFast || kind == kZero || kind == kCutHeld || kind == kTiny;
          if (BUFST)
            __builtin_amdgcn_raw_buffer_store_b128(v[i], image_rsrc, (int)(stores ? (uint32_t)(ip[i] - cimg) : kNoStore), 0,
                                                   kStorePolicySc0Sc1Nt);
          else if (stores)
            st16_aligned<NTS>(ip[i], v[i]);
        }
      } else {
#pragma unroll
        for (int i = 0; i < UNROLL; ++i) {
          const uint32_t kind = how[i] & kKind;
          if (kind == kFast) {
            st16_any<NTS>(sp[i], v[i]);
          } else if (kind == kCut) {
            // each part as at most four pieces of 8, 4, 2 and 1 bytes: exactly the bytes of the view
            const uint32_t k = (how[i] >> 8) & 0xFFu, q = how[i] >> 24;
            const bool last = how[i] & kLast;
            store_cut(sp[i], sp[i] + k + (g->pitch[q] - g->run[q]), k, v[i], last ? k : 16u);
          } else if (kind == kTiny) {
            store_low_bytes(sp[i], v[i], how[i] >> 8);
          }
        }
      }
      // Gather: a thread's further cut units, one after the other: the first k bytes end their run, the rest
      // start the next one or are padding when the payload ends there; both parts come from 16-byte loads
      // that lie wholly inside their runs.
      if (PACK && UNROLL > 1) {
#pragma unroll
        for (int i = 0; i < UNROLL; ++i)
          if ((how[i] & kKind) == kCut) {
            const uint32_t k = (how[i] >> 8) & 0xFFu, q = how[i] >> 24;
            const u32x4 va = ld16_any<NTL>(sp[i] + k - 16);
            u32x4 vb = u32x4{0, 0, 0, 0};
            if (!(how[i] & kLast)) vb = ld16_any<NTL>(sp[i] + k + (g->pitch[q] - g->run[q]));
            st16_aligned<NTS>(ip[i], splice(va, vb, 16u - k));
          }
      }
      // the rare rest (runs shorter than 16 bytes, views with several outer dimensions): a loop over a wavefront's units
      // that has each routine in the kernel once (move_unit, inlined for each of four units, takes 102 registers in the
      // scatter, which is launched for six wavefronts per SIMD: 20 MB of tensors of 1 KiB beside a view, 2048
      // work-groups, 15.7 us instead of 11.4)
      uint32_t slow = 0;
#pragma unroll
      for (int i = 0; i < UNROLL; ++i) slow |= __ballot((how[i] & kKind) == kSlow) ? 1u << i : 0u;
      const auto rest = [&](uint32_t what, uint32_t off) {  // off: the unit's place behind cb
        const uint32_t q = what >> 24;
        const uint32_t meta = (what & kKind) == kSlow ? g->meta[q] : 0u;
        const uint64_t by_lanes = __ballot(meta & DS_HOT_LANES);
        if (by_lanes)
          move_by_lanes<PACK>(a, bt, cb, cimg, by_lanes, q, off);
        if ((what & kKind) == kSlow && !(meta & DS_HOT_LANES))
          move_unit<PACK, NTL, NTS>(a.tiles + bt + q, a.hot[bt + q].img_off, cb + off, cimg + off);
      };
      if (UNROLL == 1) {
        if (slow) rest(how[0], (uint32_t)(ip[0] - cimg));
        continue;
      }
#pragma unroll 1
      for (; slow; slow &= slow - 1) {
        const int s = __builtin_ctz(slow);
        uint32_t what = how[0];
        uint32_t off = (uint32_t)(ip[0] - cimg);
#pragma unroll
        for (int i = 1; i < UNROLL; ++i)
          if (i == s) {
            what = how[i];
            off = (uint32_t)(ip[i] - cimg);
          }
        rest(what, off);
      }
    }
    uint64_t big_mask = UNROLL > 1 && NT * UNROLL >= kBigUnits ? g->big_mask : 0;
    while (big_mask) {
      const uint32_t p = (uint32_t)__builtin_ctzll(big_mask);
      big_mask &= big_mask - 1;
      const uint32_t t = bt + p;
      const uint64_t tb = a.hot[t].img_off, te = a.hot[t + 1].img_off;
      const uint64_t lo2 = tb > cb ? tb : cb, hi2 = te < ce ? te : ce;
      move_tile_direct<PACK, NT, UNROLL, NTL, NTS>(a.tiles + t, tb, lo2, hi2, a.img, a.img_lo);
    }
  }
}

// ---- chunks of several contiguous tiles ---------------------------------------------------------------------
// One chunk, whole work-group, every tile of it one contiguous run (tables of small tensors, and the chunks between
// two large ones).  The tiles' ranges follow each other in the image without a gap, so unit u of the chunk IS the
// 16 bytes at 16u: no scan over unit counts, only a binary search over where the tiles begin, as deep as the chunk
// has tiles.  And one load per unit serves all kinds: a unit cut by the end of its payload is the tile's last 16
// bytes, moved down by the bytes that were read before it.
// Bound by latency (record -> descriptors -> data) and instruction issue: see the measurements at ds_move_kernel.
struct MultiLds {
  uint64_t src[kMultiTiles];    // address of the tile's (clipped) start
  uint32_t begin[kMultiTiles];  // that start, relative to the chunk's clipped start
  uint32_t rem[kMultiTiles];    // payload bytes from there on (clamped to 2^30) | kWholeBelow16
};
constexpr uint32_t kWholeBelow16 = 1u << 31;  // the tile has less than 16 bytes: nothing to read a unit from

template <bool PACK, int NT, int UNROLL, bool NTL, bool NTS, bool BUFST, bool WHOLE>
__device__ __forceinline__ void multi_chunk(const MoveArgs &a, uint64_t c, uint32_t piece, uint32_t t0, uint32_t t1,
                                            MultiLds *g) {
  const uint32_t tid = threadIdx.x;
  uint64_t cb, ce;
  if (!piece_range<WHOLE, NT * UNROLL * 16>(a, c, piece, cb, ce)) return;
  uint8_t *const cimg = a.img + (cb - a.img_lo);
  const uint32_t size = (uint32_t)(ce - cb), n = t1 - t0 + 1;
  __syncthreads();  // readers of the previous chunk are done
  for (uint32_t i = tid; i < n; i += NT) {
    const DsTileHot *h = a.hot + t0 + i;
    const uint64_t tb = h->img_off, nbytes = h->nbytes;
    const uint64_t b0 = cb > tb ? cb - tb : 0;  // byte of the tile at which its clipped range starts
    uint64_t rem = nbytes > b0 ? nbytes - b0 : 0;
    if (rem > (1ull << 30)) rem = 1ull << 30;
    g->src[i] = h->src + b0;
    g->begin[i] = (uint32_t)(tb + b0 - cb);  // beyond the chunk's end for tiles behind the clipped range: never found
    g->rem[i] = (uint32_t)rem | (nbytes < 16 ? kWholeBelow16 : 0u);
  }
  __syncthreads();
  uint32_t p[UNROLL], d[UNROLL], rem[UNROLL];
  const uint8_t *sp[UNROLL];
#pragma unroll
  for (int i = 0; i < UNROLL; ++i) p[i] = 0;
  // the last tile that begins at or before the unit
  for (uint32_t step = 1u << (31 - __builtin_clz(n)); step > 0; step >>= 1) {
#pragma unroll
    for (int i = 0; i < UNROLL; ++i) {
      const uint32_t q = p[i] + step;
      if (q < n && g->begin[q] <= 16u * (i * NT + tid)) p[i] = q;
    }
  }
#pragma unroll
  for (int i = 0; i < UNROLL; ++i) {
    d[i] = 16u * (i * NT + tid) - g->begin[p[i]];
    rem[i] = g->rem[p[i]];
    sp[i] = (const uint8_t *)g->src[p[i]] + d[i];
  }
  u32x4 v[UNROLL];
  if (PACK) {
    uint32_t s[UNROLL];  // by how much the 16 bytes read lie before the unit; 16 = nothing of it is payload
#pragma unroll
    for (int i = 0; i < UNROLL; ++i) {
      const uint32_t whole = rem[i] & ~kWholeBelow16;
      s[i] = d[i] + 16u > whole ? d[i] + 16u - whole : 0u;
      if (s[i] > 16u || (rem[i] & kWholeBelow16)) s[i] = 16u;
      // lanes with nothing to read load the table's first bytes, so that no load hangs on a condition
      v[i] = ld16_any<NTL>(s[i] < 16u ? sp[i] - s[i] : (const uint8_t *)(a.hot + t0));
    }
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    __amdgpu_buffer_rsrc_t image_rsrc;
    if (BUFST) image_rsrc = __builtin_amdgcn_make_buffer_rsrc(cimg, 0, (int)size, 0x00020000);
#pragma unroll
    for (int i = 0; i < UNROLL; ++i) {
      if (__ballot(s[i] != 0)) {
        const u32x4 cut = splice(v[i], u32x4{0, 0, 0, 0}, s[i] & 15u);
        if (s[i] != 0) v[i] = s[i] < 16u ? cut : u32x4{0, 0, 0, 0};
        if ((rem[i] & kWholeBelow16) && d[i] < 16u) v[i] = load_low_bytes(sp[i], rem[i] & 15u);
      }
    }
#pragma unroll
    for (int i = 0; i < UNROLL; ++i) {
      const uint32_t off = 16u * (i * NT + tid);
      if (BUFST) __builtin_amdgcn_raw_buffer_store_b128(v[i], image_rsrc, (int)off, 0, kStorePolicySc0Sc1Nt);
      else if (off < size) st16_aligned<NTS>(cimg + off, v[i]);
    }
  } else {
#pragma unroll
    for (int i = 0; i < UNROLL; ++i) {
      const uint32_t off = 16u * (i * NT + tid);
      v[i] = ld16_aligned<NTL>(cimg + (off < size ? off : size - 16u));
    }
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
#pragma unroll
    for (int i = 0; i < UNROLL; ++i) {
      const uint32_t whole = rem[i] & ~kWholeBelow16;
      if (16u * (i * NT + tid) < size && d[i] < whole) {
        if (d[i] + 16u <= whole) st16_any<NTS>((uint8_t *)sp[i], v[i]);
        else store_low_bytes((uint8_t *)sp[i], v[i], whole - d[i]);
      }
    }
  }
}

// ---- the lean path -----------------------------------------------------------
// BUFST: the gather writes the image through buffer stores with the cache policy "sc0 sc1 nt"
// (write-through, streaming).  Measured on a plain copy of this shape: 6.25 TB/s against 6.07 TB/s with
// "nt" global stores and 5.88 TB/s with plain ones.  The buffer form is used because the compiler has an
// intrinsic with a cache-policy operand for it (and none for global stores); the resource covers exactly
// the work-group's chunk, so an out-of-range store would be dropped by the hardware.

// A record, in one scalar load: the table is constant while the kernel runs.  Through an ordinary pointer the compiler
// reads it in two vector loads, the second behind the first's answer.
__device__ __forceinline__ DsChunkRec load_rec(const DsChunkRec *recs, uint64_t i) {
  typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
  const u32x8 w = *(const __attribute__((address_space(4))) u32x8 *)(uintptr_t)(recs + i);
  return DsChunkRec{w[0] | (uint64_t)w[1] << 32, w[2] | (uint64_t)w[3] << 32, w[4], w[5], w[6], w[7]};
}
__device__ __forceinline__ uint32_t load_id(const uint32_t *ids, uint64_t i) {
  return *(const __attribute__((address_space(4))) uint32_t *)(uintptr_t)(ids + i);
}

// Moves a lean chunk, or its piece of NT * UNROLL units from byte `piece` on, which is at imgp in the image buffer.
template <bool PACK, int NT, int UNROLL, bool NTL, bool NTS, bool BUFST>
__device__ __forceinline__ void lean_move(const DsChunkRec &r, uint8_t *imgp, uint32_t piece) {
  const uint32_t tid = threadIdx.x;
  __amdgpu_buffer_rsrc_t image_rsrc;
  if (PACK && BUFST) image_rsrc = __builtin_amdgcn_make_buffer_rsrc(imgp, 0, NT * UNROLL * 16, 0x00020000);
  u32x4 v[UNROLL];
  if ((r.kind & 0xFFu) == DS_CHUNK_CONTIG) {
    uint8_t *s = reinterpret_cast<uint8_t *>(r.addr) + piece;
    // (the scatter keeps "nt" global stores on the tensor side: the write-through buffer stores that serve
    // the image so well cost it 3 % on the Llama ranks and 10 % on the fragmentation set, measured)
    if (PACK && (r.kind & DS_CHUNK_REALIGN)) {
      // The tensor side is at an odd address: a 16-byte load there costs about twice an aligned one.  Every
      // lane loads the ALIGNED unit that holds the first byte of its image unit and takes the rest from
      // the unit of the lane above it (of the same wavefront: the last lane loads that unit itself); the
      // plan sets the flag only where those units lie inside the tensor.
      const uint32_t m = (uint32_t)r.addr & 15u;
      uint8_t *base = s - m;
      const bool last_lane = (tid & (kWave - 1)) == kWave - 1;
      u32x4 a[UNROLL], e[UNROLL];
#pragma unroll
      for (int i = 0; i < UNROLL; ++i) a[i] = ld16_aligned<NTL>(base + 16u * (i * NT + tid));
#pragma unroll
      for (int i = 0; i < UNROLL; ++i) {
        e[i] = u32x4{0, 0, 0, 0};
        if (last_lane) e[i] = ld16_aligned<NTL>(base + 16u * (i * NT + tid) + 16u);
      }
#pragma unroll
      for (int i = 0; i < UNROLL; ++i) {
        u32x4 up = u32x4{lane_above(a[i].x), lane_above(a[i].y), lane_above(a[i].z), lane_above(a[i].w)};
        if (last_lane) up = e[i];
        v[i] = splice(a[i], up, m);
      }
    } else {
#pragma unroll
      for (int i = 0; i < UNROLL; ++i) {
        const uint32_t off = 16u * (i * NT + tid);
        v[i] = PACK ? ld16_any<NTL>(s + off) : ld16_aligned<NTL>(imgp + off);
      }
    }
#pragma unroll
    for (int i = 0; i < UNROLL; ++i) {
      const uint32_t off = 16u * (i * NT + tid);
      if (PACK && BUFST) __builtin_amdgcn_raw_buffer_store_b128(v[i], image_rsrc, (int)off, 0, kStorePolicySc0Sc1Nt);
      else if (PACK) st16_aligned<NTS>(imgp + off, v[i]);
      else st16_any<NTS>(s + off, v[i]);
    }
  } else {
    // DS_CHUNK_ROWS: runs of r.run >= 16 bytes, r.pitch apart.  A unit that lies in one
    // run is one access.  A unit cut by the end of a run takes its first k bytes from
    // the end of that run and the other 16-k from the start of the next one; on the
    // gather side both come from 16-byte loads that lie wholly inside their runs
    // (the last 16 bytes of the one, the first 16 of the other), so nothing outside
    // the view is read; on the scatter side each part is stored as at most four pieces
    // of 8, 4, 2 and 1 bytes, exactly the bytes of the view.
    uint8_t *p[UNROLL];
    uint32_t cut[UNROLL];  // k, or 0 if the unit is not cut
    u32x4 w[UNROLL];       // gather: the first 16 bytes of the next run, for cut units
    // One division for the thread's first unit; its other units are NT*16 bytes further on each,
    // and the plan has divided that step by the run length already (r.tile = quotient << 16 | rest).
    const uint32_t step_q = r.tile >> 16, step_r = r.tile & 0xFFFFu;
    const uint32_t tt0 = r.col0 + piece + 16u * tid;  // < 2^31 + 2^15
    uint32_t q = tt0 / r.run;
    uint32_t col = tt0 - q * r.run;
#pragma unroll
    for (int i = 0; i < UNROLL; ++i) {
      const uint32_t off = 16u * (i * NT + tid);
      uint8_t *row = reinterpret_cast<uint8_t *>(r.addr + (uint64_t)q * r.pitch);
      p[i] = row + col;
      cut[i] = col + 16u > r.run ? r.run - col : 0u;
      if (PACK) {
        // all loads are issued before any of them is used: no wait inside this loop
        v[i] = ld16_any<NTL>(cut[i] ? row + r.run - 16u : p[i]);
        if (cut[i]) w[i] = ld16_any<NTL>(row + r.pitch);
      } else {
        v[i] = ld16_aligned<NTL>(imgp + off);
      }
      q += step_q;
      col += step_r;
      if (col >= r.run) {
        col -= r.run;
        ++q;
      }
    }
    if (PACK) {
#pragma unroll
      for (int i = 0; i < UNROLL; ++i)
        if (cut[i]) v[i] = splice(v[i], w[i], 16u - cut[i]);
    }
#pragma unroll
    for (int i = 0; i < UNROLL; ++i) {
      const uint32_t off = 16u * (i * NT + tid);
      if (PACK && BUFST) {
        __builtin_amdgcn_raw_buffer_store_b128(v[i], image_rsrc, (int)off, 0, kStorePolicySc0Sc1Nt);
      } else if (PACK) {
        st16_aligned<NTS>(imgp + off, v[i]);
      } else if (cut[i] == 0) {
        st16_any<NTS>(p[i], v[i]);
      } else {
        store_cut(p[i], p[i] + cut[i] + (r.pitch - r.run), cut[i], v[i]);
      }
    }
  }
}

// Moves a chunk of kind DS_CHUNK_DIMS, or its piece of NT * UNROLL units from byte `piece` on, which is at imgp in the image
// buffer.  As lean_move does with rows, but for the address of a run, which takes a division per outer dimension; the tile's
// extents and strides are in scalar registers.  Through the general path (LDS, the tile's descriptor per lane, one unit after
// the other) a view of three dimensions was slower with one unit per thread than with four.  64 MB in runs of 256 bytes,
// gather / scatter, four units and one through the general path 63.5 / 53.8 and 60.1 / 60.2 us, now 26.5 / 29.3; 5 GB of
// runs of 2 KiB 4095 / 3622, 4149 / 3943, now 1606 / 1704.
template <bool PACK, int NT, int UNROLL, bool NTL, bool BUFST>
__device__ __forceinline__ void dims_move(const DsChunkRec &r, const DsTile *tiles, uint8_t *imgp, uint32_t piece) {
  const uint32_t tid = threadIdx.x;
  const DS_CONSTANT DsTile *t = (const DS_CONSTANT DsTile *)(uintptr_t)(tiles + r.tile);
  const auto run_at = [&](uint32_t row) {
    uint64_t x = t->src;
#pragma unroll 1
    for (uint32_t j = t->n_outer - 1; j > 0; --j) {
      const uint32_t extent = (uint32_t)t->extent[j], rows = row / extent;
      x += (row - rows * extent) * t->stride[j];
      row = rows;
    }
    return reinterpret_cast<uint8_t *>(x + row * t->stride[0]);
  };
  __amdgpu_buffer_rsrc_t image_rsrc;
  if (PACK && BUFST) image_rsrc = __builtin_amdgcn_make_buffer_rsrc(imgp, 0, NT * UNROLL * 16, 0x00020000);
  uint8_t *p[UNROLL], *next[UNROLL];  // the unit; the run behind its own, if it goes on there
  uint32_t cut[UNROLL];               // how much of it is in its own run, or 0 if all is
  u32x4 v[UNROLL], w[UNROLL];
#pragma unroll
  for (int i = 0; i < UNROLL; ++i) {
    const uint32_t off = 16u * (i * NT + tid), at = (uint32_t)r.pitch + piece + off;  // < 2^31 + 2^14
    const uint32_t rows = at / r.run, col = at - rows * r.run, row = (uint32_t)r.addr + rows;
    uint8_t *const run = run_at(row);
    p[i] = run + col;
    cut[i] = col + 16u > r.run ? r.run - col : 0u;
    if (cut[i]) next[i] = run_at(row + 1);
    if (PACK) {
      v[i] = ld16_any<NTL>(cut[i] ? run + r.run - 16u : p[i]);
      if (cut[i]) w[i] = ld16_any<NTL>(next[i]);
    } else {
      v[i] = ld16_aligned<NTL>(imgp + off);
    }
  }
#pragma unroll
  for (int i = 0; i < UNROLL; ++i) {
    const uint32_t off = 16u * (i * NT + tid);
    if (PACK) {
      if (cut[i]) v[i] = splice(v[i], w[i], 16u - cut[i]);
      if (BUFST) __builtin_amdgcn_raw_buffer_store_b128(v[i], image_rsrc, (int)off, 0, kStorePolicySc0Sc1Nt);
      else st16_aligned<true>(imgp + off, v[i]);
    } else if (cut[i]) {
      store_cut(p[i], next[i], cut[i], v[i]);
    } else {
      st16_any<true>(p[i], v[i]);
    }
  }
}

// Number of lean work items of a launch; item ci takes one lean chunk, whole work-group.
__device__ __forceinline__ uint32_t lean_items(const LeanArgs &a) { return a.xcd_span ? a.xcd_span * 8u : a.n_pieces; }

// Work item ci of a launch: moves its chunk if the chunk is lean and returns 0; for any other it moves nothing, says
// which chunk and tiles (c, t0, t1) and returns the chunk's kind: the caller sends it down its path (one call site
// each, so that these paths are in the kernel once).
// WALKS: the launch has fewer work-groups than work items.  A work-group's next record is then read with vector loads: as a
// scalar load, 300 MB in one tensor with 1024 work-groups took 121 us (scatter 119) instead of 110 (107), a 4 x smaller rank
// 85 (89) instead of 76 (75).  Where every work-group has one item the scalar load is the faster one (20 000 fragments of
// 2.5 GB 496 / 513 us).
// BLOCKS is a template parameter and not a test of `ids`: the test alone made a 23 MB gather 0.9 us slower.
template <bool PACK, int NT, int UNROLL, bool NTL, bool NTS, bool BUFST, int BLOCKS, bool WHOLE, bool WALKS>
__device__ __forceinline__ uint32_t lean_chunk(const LeanArgs &a, uint32_t ci, uint32_t pieces_log2, uint64_t &c_gen,
                                               uint32_t &piece, uint32_t &t0, uint32_t &t1) {
  // Work-groups are dealt to the 8 XCDs round-robin (work-group i runs on XCD i mod 8).  Chunk
  // numbers are permuted so that each XCD walks ONE contiguous eighth of the range instead of every
  // eighth chunk: measured +1.5 % (7B rank) to +5 % (fragmentation set) on the gather and +4 to +8 %
  // on the scatter.
  uint32_t cm = ci;
  if (a.xcd_span) {
    cm = (ci & 7u) * a.xcd_span + (ci >> 3);
    if (cm >= a.n_pieces) return 0;
  }
  if (!WHOLE) piece = (cm & ((1u << pieces_log2) - 1)) * (NT * UNROLL * 16);  // offset inside the chunk
  const uint32_t rec = a.c_lo + (WHOLE ? cm : cm >> pieces_log2);
  const DsChunkRec r = WALKS ? a.recs[rec] : load_rec(a.recs, rec);
  const uint32_t c = BLOCKS != kListed ? rec : WALKS ? a.ids[rec] : load_id(a.ids, rec);
  const uint32_t kind = r.kind & 0xFF;  // bits 8.. hold log2(itemsize)
  if (BLOCKS == kBeside && kind == DS_CHUNK_PERM) return 0;
  if (kind >= DS_CHUNK_GENERAL) {
    // its record names the tiles it holds: one load away from them, and in place among its neighbours
    c_gen = c;
    t0 = r.tile;
    t1 = r.tile + r.col0;
    return kind;
  }
  const uint32_t from = WHOLE ? 0u : piece;
  lean_move<PACK, NT, UNROLL, NTL, NTS, BUFST>(r, a.img + (((uint64_t)c << a.chunk_log2) - a.img_lo) + from, from);
  return 0;
}

// The tiles t0 .. t1 of a chunk that is cut by the range.
__device__ __forceinline__ void cut_chunk_tiles(const MoveArgs &a, uint64_t c, uint32_t &t0, uint32_t &t1) {
  uint64_t c_end = (c + 1) << a.chunk_log2;
  if (c_end > a.total) c_end = a.total;
  t0 = a.first_tile[c];
  t1 = a.first_tile[c + 1];
  if (a.hot[t1].img_off >= c_end) --t1;  // that tile starts where this chunk ends
}

// Both paths in one launch: work item i takes whole chunk number i of the range (in the XCD-contiguous
// order) down the path its record names, so a general chunk is moved in place, among its neighbours in the
// image, one record load away from its tiles; the at most two chunks cut by the ends of the range follow
// as work items of their own.  History, measured on the gather: lean kernel then general kernel in two
// launches cost the 7B rank a launch gap plus the general kernel's 9 us (5.78 TB/s in the timed region
// against 6.17 now); the general kernel on a side stream beside the lean one gave the fragmentation set
// 5.30 -> 5.54 TB/s, one launch 5.85 TB/s.
//
// A work-group takes one piece of a chunk, 256 threads x UNROLL units, with at most WAVES wavefronts per SIMD (the
// attribute makes the compiler pad the register allocation).
//   gather, UNROLL 4 and WAVES 4: 64 KB in flight, and few work-groups keep the addresses in a compact window of
//     HBM (five wavefronts -0.8 % on the 7B and 70B ranks, eight -4 %, three or fewer -9 %).
//   gather of plans of mostly general chunks, WAVES 6: that path is bound by its chain of dependent loads (+8 to +10 %
//     on tables of tiny tensors against four).
//   scatter, UNROLL 2 and WAVES 6 (a piece of 8 KiB, 48 KB in flight), or as the gather: see launch_scatter.
// PATH kMulti is the instantiation for plans of contiguous shards only, most chunks of which hold several of them:
// no chunk takes the general path, and multi_chunk's registers (gather 78, scatter 32) allow six and eight wavefronts.
// 24 000 tensors of 16 bytes to 16 KiB (58 MB), with non-temporal loads: gather 24.7 us against 29.1 through the general
// path, scatter 23.9 against 26.6; with ordinary loads (kCachedBytes) 19.1 and 18.8, a plain copy of it takes 16.6.  One
// unit per thread 19.8 and 21.0 (147 MB: 56.4 and 55.2, as it is 54.0 and 55.4), ordinary stores 26.6 and 26.9.
enum : int { kEvery = 0, kMulti = 1 };
// Does a work-group of so many units take whole chunks (else pieces of them)?
constexpr bool takes_whole_chunks(bool pack, int units) { return units >= (pack ? 512 : 1024); }
template <bool PACK, int NT, int UNROLL, bool NTL, bool NTS, bool BUFST, int WAVES, int BLOCKS, int PATH, bool WALKS>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(1, WAVES))) void ds_move_kernel(
    const DsChunkRec *recs, const uint32_t *ids, uint8_t *img, uint64_t img_lo, uint32_t chunk_log2, uint32_t c_lo,
    uint32_t n_pieces, uint32_t xcd_span, MoveArgs ma) {
  const LeanArgs la = {recs, ids, img, img_lo, chunk_log2, c_lo, n_pieces, xcd_span};
  __shared__ typename std::conditional<PATH == kMulti, MultiLds, GenLds>::type s_tab;
  const uint32_t n_lean = lean_items(la);
  constexpr bool WHOLE = takes_whole_chunks(PACK, NT * UNROLL);
  const uint32_t pieces_log2 = WHOLE ? 0 : ma.n_extra >> 8;
  const uint32_t n_iter = n_lean + (WHOLE ? ma.n_extra : (ma.n_extra & 0xFFu) << pieces_log2);
  for (uint32_t wi = blockIdx.x; wi < n_iter; wi += gridDim.x) {
    uint64_t c = 0;
    uint32_t piece = 0, t0 = 0, t1 = 0;
    uint32_t kind = DS_CHUNK_GENERAL;
    if (wi < n_lean) {
      kind = lean_chunk<PACK, NT, UNROLL, NTL, NTS, BUFST, BLOCKS, WHOLE, WALKS>(la, wi, pieces_log2, c, piece, t0, t1);
    } else {
      // (a piece of) a chunk cut by the range, whatever the chunk's kind: these paths clip to the range
      const uint32_t x = wi - n_lean;
      c = ma.extra[x >> pieces_log2];
      piece = (x & ((1u << pieces_log2) - 1)) * (NT * UNROLL * 16);
      cut_chunk_tiles(ma, c, t0, t1);
    }
    if constexpr (PATH == kMulti) {
      if (kind) multi_chunk<PACK, NT, UNROLL, NTL, NTS, BUFST, WHOLE>(ma, c, piece, t0, t1, &s_tab);
    } else {
      constexpr int PASS = PATH == kEvery && WHOLE ? 4 : UNROLL;
      if (kind)
        general_chunk<PACK, NT, PASS, NTL, NTS, BUFST, BLOCKS, WHOLE>(ma, c, piece, t0, t1, &s_tab);
    }
  }
}

// The same, one unit per thread and one piece of 4 KiB per work-group, for plans of 16 KiB chunks: what a default call
// launches unless most chunks hold several contiguous tensors (multi_chunk).  With one load and one store per wavefront
// the lean path is bound by HBM as long as eight wavefronts per SIMD fit (64 registers: hence no loop over work items,
// whose constants the compiler keeps in registers, move_runs, and a scan without LDS) and a wavefront has done its work in the 700 cycles
// that its 1 KiB takes its SIMD's share of HBM: the record in one scalar load, nothing else in front of the data.  (With
// the record in two vector loads, one behind the other, the 7.6 GB gather took 3137 us.)  Measured, four units per thread
// and four wavefronts (scatter: two and six) before / now: gather of a 70B rank (7.6 GB) 2392 / 2280 us, scatter of a 7B
// rank (1.5 GB) 490 / 473, 20 000 fragments (7.5 GB) 2488 / 2356, a 23 MB state 10.9 / 9.1 and scatter 11.4 / 8.9 (with the
// ordinary loads of small images; non-temporal 10.0 and 10.6), 475 fragments with many rows (1 MB) 8.0 / 6.3.
// Work-groups of 512 and 1024 threads measure the same on large tensors and 3 to 5 % slower on fragments.
// (DIMS: the plan has chunks of that kind.  The test alone makes the compiler move scalar registers to and fro in front of
// every chunk: a 210 MB rank 65.9 us instead of 64.7.)
template <bool PACK, bool NTL, int BLOCKS, bool DIMS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8, 8))) void ds_unit_kernel(
    const DsChunkRec *recs, const uint32_t *ids, uint8_t *img0, uint32_t n, uint32_t span, uint32_t c_lo, MoveArgs ma) {
  __shared__ GenLds s_tab;
  const uint32_t wi = blockIdx.x, cm = (wi & 7u) * span + (wi >> 3);
  uint64_t c;
  uint32_t piece, t0, t1;
  if (wi < span * 8u) {
    if (cm >= n) return;
    const uint32_t rec = c_lo + cm / kUnitPieces;
    piece = cm % kUnitPieces * 4096;
    const DsChunkRec r = load_rec(recs, rec);
    c = BLOCKS == kListed ? load_id(ids, rec) : rec;
    const uint32_t kind = r.kind & 0xFFu;
    if (kind < DS_CHUNK_GENERAL) {
      lean_move<PACK, 256, 1, NTL, true, PACK>(r, img0 + (c << 14) + piece, piece);
      return;
    }
    if (DIMS && kind == DS_CHUNK_DIMS) {
      dims_move<PACK, 256, 1, NTL, PACK>(r, ma.tiles, img0 + (c << 14) + piece, piece);
      return;
    }
    if (BLOCKS == kBeside && kind == DS_CHUNK_PERM) return;
    t0 = r.tile;
    t1 = r.tile + r.col0;
  } else {
    const uint32_t x = wi - span * 8u;
    c = ma.extra[x / kUnitPieces];
    piece = x % kUnitPieces * 4096;
    cut_chunk_tiles(ma, c, t0, t1);
  }
  general_chunk<PACK, 256, 1, NTL, true, PACK, BLOCKS, false>(ma, c, piece, t0, t1, &s_tab);
}

template <bool PACK, bool NTL, int BLOCKS, bool DIMS>
int launch_units(const LeanArgs &la, const MoveArgs &ma, hipStream_t stream) {
  const uint32_t n = la.n_pieces * kUnitPieces, span = (n + 7) / 8, grid = span * 8 + ma.n_extra * kUnitPieces;
  if (grid == 0) return DS_OK;
  hipLaunchKernelGGL((ds_unit_kernel<PACK, NTL, BLOCKS, DIMS>), dim3(grid), dim3(256), 0, stream, la.recs, la.ids,
                     la.img - la.img_lo, n, span, la.c_lo, ma);
  DS_HIP_TRY(hipGetLastError());
  return DS_OK;
}

template <bool PACK, int BLOCKS>
int launch_units(const ds_plan *plan, const LeanArgs &la, const MoveArgs &ma, hipStream_t stream) {
  const bool dims = plan->n_dims != 0;
  if (plan->total_bytes <= kCachedBytes)
    return dims ? launch_units<PACK, false, BLOCKS, true>(la, ma, stream) : launch_units<PACK, false, BLOCKS, false>(la, ma, stream);
  return dims ? launch_units<PACK, true, BLOCKS, true>(la, ma, stream) : launch_units<PACK, true, BLOCKS, false>(la, ma, stream);
}

constexpr uint32_t kMaxGrid = 1u << 23;  // work-groups of 256: a launch has less than 2^32 threads

template <bool PACK, int NT, int UNROLL, bool NTL, bool NTS, bool BUFST, int WAVES, int BLOCKS, int PATH>
int launch_pieces(LeanArgs la, MoveArgs ma, uint32_t grid_limit, hipStream_t stream) {
  const uint32_t pieces_log2 = la.chunk_log2 - (4 + __builtin_ctz(NT * UNROLL));
  la.n_pieces <<= pieces_log2;  // chunks so far
  la.xcd_span = ds_cfg_variant() == 3 ? 0 : (la.n_pieces + 7) / 8;
  const uint64_t items = (uint64_t)(la.xcd_span ? la.xcd_span * 8 : la.n_pieces) + (ma.n_extra << pieces_log2);
  uint64_t grid = items;
  if (grid == 0) return DS_OK;
  if (!takes_whole_chunks(PACK, NT * UNROLL)) ma.n_extra |= pieces_log2 << 8;
  else if (pieces_log2) return DS_EINVAL;
  if (grid_limit && grid > grid_limit) grid = grid_limit;
  if (grid > kMaxGrid * 256 / NT) grid = kMaxGrid * 256 / NT;
  // (not for plans of small tensors, which are never launched so, nor for the policies of variants 1 and 2)
  constexpr bool kWalks = PATH == kEvery && NTL && BUFST == PACK;
  if (kWalks && grid < items)
    hipLaunchKernelGGL((ds_move_kernel<PACK, NT, UNROLL, NTL, NTS, BUFST, WAVES, BLOCKS, PATH, kWalks>),
                       dim3((uint32_t)grid), dim3(NT), 0, stream, la.recs, la.ids, la.img, la.img_lo, la.chunk_log2, la.c_lo,
                       la.n_pieces, la.xcd_span, ma);
  else
    hipLaunchKernelGGL((ds_move_kernel<PACK, NT, UNROLL, NTL, NTS, BUFST, WAVES, BLOCKS, PATH, false>),
                       dim3((uint32_t)grid), dim3(NT), 0, stream, la.recs, la.ids, la.img, la.img_lo, la.chunk_log2, la.c_lo,
                       la.n_pieces, la.xcd_span, ma);
  DS_HIP_TRY(hipGetLastError());
  return DS_OK;
}

// The gather: a chunk per work-group.  (Pieces in its kernel, though one per chunk, cost the 23 MB gather 0.3 us.)
template <bool NTL, bool NTS, bool BUFST, int WAVES = 4, int BLOCKS = kAlone, int PATH = kEvery>
int launch_gather(const LeanArgs &la, const MoveArgs &ma, uint32_t grid_limit, hipStream_t stream) {
  switch (la.chunk_log2) {
    case 13: return launch_pieces<true, 256, 2, NTL, NTS, BUFST, WAVES, BLOCKS, PATH>(la, ma, grid_limit, stream);
    case 14: return launch_pieces<true, 256, 4, NTL, NTS, BUFST, WAVES, BLOCKS, PATH>(la, ma, grid_limit, stream);
    case 15: return launch_pieces<true, 256, 8, NTL, NTS, BUFST, WAVES, BLOCKS, PATH>(la, ma, grid_limit, stream);
    default: return DS_EINVAL;
  }
}

// The scatter, in whole chunks at four wavefronts per SIMD or in pieces of 8 KiB at six (ds_plan::scatter_in_pieces).
// Plans of mostly general chunks keep whole chunks, whose tiles are looked up once, at six (20 MB of tensors of 1 KiB
// beside a view, 2048 work-groups: 11.3 us, at four 15.7).
template <bool NTL, bool NTS, int BLOCKS = kAlone, int PATH = kEvery>
int launch_scatter(const ds_plan *plan, bool few, bool mostly_general, const LeanArgs &la, const MoveArgs &ma,
                   uint32_t grid_limit, hipStream_t stream) {
  if constexpr (PATH == kMulti) {
    return launch_pieces<false, 256, 2, NTL, NTS, false, 8, BLOCKS, PATH>(la, ma, grid_limit, stream);
  } else {
    const bool large = la.chunk_log2 == 15;
    if (la.chunk_log2 > 13 && mostly_general)
      return large ? launch_pieces<false, 256, 8, NTL, NTS, false, 6, BLOCKS, PATH>(la, ma, grid_limit, stream)
                   : launch_pieces<false, 256, 4, NTL, NTS, false, 6, BLOCKS, PATH>(la, ma, grid_limit, stream);
    if (la.chunk_log2 > 13 && (few || !plan->scatter_in_pieces((uint64_t)la.n_pieces << (la.chunk_log2 - 14))))
      return large ? launch_pieces<false, 256, 8, NTL, NTS, false, 4, BLOCKS, PATH>(la, ma, grid_limit, stream)
                   : launch_pieces<false, 256, 4, NTL, NTS, false, 4, BLOCKS, PATH>(la, ma, grid_limit, stream);
    return launch_pieces<false, 256, 2, NTL, NTS, false, 6, BLOCKS, PATH>(la, ma, grid_limit, stream);
  }
}

// The chunks of a plan whose views with short runs another launch moves in blocks.
template <int BLOCKS>
int launch_beside_blocks(const ds_plan *plan, bool pack, bool few, bool mostly_general, const LeanArgs &la,
                         const MoveArgs &ma, uint32_t grid_limit, hipStream_t stream) {
  if (!pack) return launch_scatter<true, true, BLOCKS>(plan, few, mostly_general, la, ma, grid_limit, stream);
  if (mostly_general) return launch_gather<true, true, true, 6, BLOCKS>(la, ma, grid_limit, stream);
  return launch_gather<true, true, true, 4, BLOCKS>(la, ma, grid_limit, stream);
}

// Plans of views and mostly chunks of several contiguous tensors (ds_plan::mostly_several), chunks of 16 KiB.
template <bool NTL, int BLOCKS>
int launch_several(bool pack, const LeanArgs &la, const MoveArgs &ma, hipStream_t stream) {
  if (pack) return launch_pieces<true, 256, 4, NTL, true, true, 6, BLOCKS, kEvery>(la, ma, 0, stream);
  return launch_pieces<false, 256, 4, NTL, true, false, 6, BLOCKS, kEvery>(la, ma, 0, stream);
}
template <int BLOCKS>
int launch_several(const ds_plan *plan, bool pack, const LeanArgs &la, const MoveArgs &ma, hipStream_t stream) {
  return plan->total_bytes <= kCachedBytes ? launch_several<false, BLOCKS>(pack, la, ma, stream)
                                           : launch_several<true, BLOCKS>(pack, la, ma, stream);
}

// ---- views with runs shorter than 16 bytes, in blocks through LDS (ds_perm.h) ---------------------------
// Bound by HBM as far as both sides have whole lines (wide blocks, ds_perm.h: 4.7 TB/s on large transpositions), else by
// the memory system's handling of parts of lines: every second column, six of every sixteen columns, whose lines the
// scatter writes in part.  A block's descriptor is read as constant memory: read through ordinary pointers, again after
// every store that might have changed it, the table of such views of perf/cases.py took 93.4 us instead of 79.3 (gather).
// That table: unit by unit 460 / 524 us, in narrow blocks 100 / 108, now 79 / 98; channels-last 14.1 / 14.5, now 10.8 /
// 13.1; every second fp32 column 10.9 / 14.4, now 10.1 / 12.8; with the blocks in stripes over the XCDs (ds_perm_order) and
// streaming loads (STREAM: images that no cache holds until the next pass) 63.2 / 68.8, with short rows and short runs in larger
// accesses (ds_perm_groups, ds_perm_runs) 61.5 / 67.2, now 57.5 / 64.0; with the lines of which views hold parts, 38 MB that the
// counters see the gather read and the scatter write, a plain copy would take 55.  Streaming loads alone are worth, us:
// gather, where no line of the tensor is another block's too (kPermOnce), bf16 4096 x 4096 62.4 / 59.5 (five of them), every
// second column 86.5 / 80.6 (ten), channels-last 75.8 / 72.1; where lines are shared they cost (bytes 4096 x 4120 68 / 81);
// the scatter's loads 62.4 / 57.9, but not beside wide blocks whose stores stay in the caches to meet their lines' other
// parts (1000 x 1007 75.4 / 82.1), and not in short rows, whose lines several blocks read (kPermImageOnce).  Images that the last-level cache holds lose (one of 33 MB 13.1 / 16.5).
// Blocks are numbered along b first: along a first costs 15 % of the gather.  LDS has room for five work-groups per CU, in
// launches without wide blocks (WIDE = false) for seven:
// 8000 squares of 24 bf16, gather / scatter, 30.4 / 32.0 with five, 27.1 / 28.8 with seven; a channels-last convolution of 46 MB
// 24.0 / 28.5 and 21.7 / 26.1; three of every eight bytes 34.1 / 42.9 and 32.9 / 43.0.
struct PermArgs {
  const DsPerm *perms;
  const DsPermItem *items;  // the launch's first block
  uint32_t n_items;
  uint32_t xcd_span;        // work-groups per XCD; 0 = work-group i takes block i
  uint32_t stripe, magic;   // the order of the blocks (DsPermOrder)
};
struct ImageArgs {
  uint8_t *img;             // points at image byte img_lo
  uint64_t img_lo, img_hi;
};

template <typename E, typename W, bool PACK, bool STREAM>
__device__ __forceinline__ void move_perm_block(const DS_PERM_TABLE DsPerm &d, const DsPermBlock &k, const ImageArgs &a, uint8_t *lds) {
  // opaque, so that nothing made of it is kept in registers (beyond 96: in scratch) across the loop over the blocks
  uint32_t tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  if (PACK) {
    ds_perm_tensor_side<E, W, true, STREAM>(d, k, lds, tid);
    __syncthreads();
    // rows that end inside a line leave its rest to another block: the line is better kept in the L2 until then
    // (bytes transposed into rows of 112: 16.1 us streaming, 12.1 us cached; rows of whole lines 16.2 and 17.7)
    // (Two loops: one loop with both stores is compiled to one store, the cached one.)
    if (d.flags & (kPermLines | kPermWide))
      ds_perm_image_store<E>(d, k, lds, a.img, a.img_lo, tid, [](uint64_t p, const DsPermUnit &v) {
        st16_aligned<true>((uint8_t *)p, u32x4{v.w[0], v.w[1], v.w[2], v.w[3]});
      });
    else
      ds_perm_image_store<E>(d, k, lds, a.img, a.img_lo, tid, [](uint64_t p, const DsPermUnit &v) {
        st16_aligned<false>((uint8_t *)p, u32x4{v.w[0], v.w[1], v.w[2], v.w[3]});
      });
  } else {
    if (STREAM && (d.flags & kPermImageOnce))
      ds_perm_image_load(d, k, lds, a.img, a.img_lo, ds_perm_apart<true>(tid), [](uint64_t p) {
        const u32x4 v = ld16_aligned<true>((const uint8_t *)p);
        return DsPermUnit{{v.x, v.y, v.z, v.w}};
      });
    else
      ds_perm_image_load(d, k, lds, a.img, a.img_lo, tid, [](uint64_t p) {
        const u32x4 v = ld16_aligned<false>((const uint8_t *)p);
        return DsPermUnit{{v.x, v.y, v.z, v.w}};
      });
    __syncthreads();
    ds_perm_tensor_side<E, W, false, STREAM>(d, k, lds, tid);
  }
}

// Item i of a launch: one block.
template <bool PACK, bool STREAM>
__device__ __forceinline__ void move_perm_item(const PermArgs &p, const ImageArgs &a, uint32_t i, uint8_t *lds) {
  const DS_PERM_TABLE DsPermItem &item = ((const DS_PERM_TABLE DsPermItem *)(uintptr_t)p.items)[i];
  const DS_PERM_TABLE DsPerm &d = ((const DS_PERM_TABLE DsPerm *)(uintptr_t)p.perms)[item.perm];
  DsPermBlock k;
  if (!ds_perm_block(d, item.tile, a.img_lo, a.img_hi, PACK, k)) return;
  switch (d.flags & 0xFFu) {
    case 0: move_perm_block<uint8_t, uint32_t, PACK, STREAM>(d, k, a, lds); break;
    case 1: move_perm_block<uint16_t, uint32_t, PACK, STREAM>(d, k, a, lds); break;
    case 2: move_perm_block<uint32_t, uint32_t, PACK, STREAM>(d, k, a, lds); break;
    default: move_perm_block<uint64_t, uint64_t, PACK, STREAM>(d, k, a, lds); break;
  }
}

template <bool PACK, bool STREAM, bool WIDE>
__global__ __launch_bounds__(256, 5) void ds_perm_kernel(const DsPerm *perms, const DsPermItem *items, uint32_t n_items,
                                                         uint32_t xcd_span, uint32_t stripe, uint32_t magic, ImageArgs image) {
  const PermArgs a = {perms, items, n_items, xcd_span, stripe, magic};
  __shared__ __attribute__((aligned(16))) uint8_t s_block[WIDE ? kPermLdsBytes : kPermNarrowBytes];
  const uint32_t n = a.xcd_span ? a.xcd_span * 8u : a.n_items;
  for (uint32_t wi = blockIdx.x; wi < n; wi += gridDim.x) {
    const uint32_t i = a.xcd_span ? ds_perm_ordered(wi, a.stripe, a.magic) : wi;
    if (i >= a.n_items) continue;
    move_perm_item<PACK, STREAM>(a, image, i, s_block);
    __syncthreads();  // the block in LDS has been used
  }
}

constexpr uint32_t kMixedChunks = 4096;  // other chunks up to which blocks and chunks share a launch
constexpr uint32_t kMixedInPieces = 640; // ... and are moved 4 KiB per work-group

// Blocks and the plan's other chunks in one launch: first the blocks, then the chunks, 16 KiB per work-group, which fill
// the chip while the last blocks end.  A second launch costs 3 us and the ramps between the two; in exchange the chunks move at
// five wavefronts per SIMD, four units per thread.  One launch / two, us, gather and scatter: the views of perf/cases.py
// (157 MB, 2048 chunks beside the blocks) 75.3 / 79.4 and 97.0 / 98.5, the same at a quarter of the columns 9.0 / 11.8 and
// 9.7 / 13.7, at a sixteenth 6.9 / 9.9; one transposed matrix of 32 KB to 8 MB beside 32 MB 14.5 to 16.7 / 16.3 to 18.9;
// beside 100 MB (6400 chunks) 40.9 / 41.5 and 40.3 / 39.3; 32 MB beside 400 MB 153.8 / 142.8 and 152.8 / 145.7.
// PIECES: up to 640 chunks, 4 KiB per work-group, one unit per thread.  All work-groups run at once then, and the launch takes as long
// as the slowest, which is a chunk where several shards meet (the general path) or of a view of several dimensions.  Such
// chunks whole, one unit per thread after the other / in pieces, us, gather and scatter: views of 592 columns of 8 bytes (10 MB)
// 11.3 / 7.2 and 10.0 / 6.5, 2160 columns of f16 (43 MB) 22.2 / 17.6 and 26.2 / 21.5; 8 MB in tensors of 65 000 bytes beside a
// view 7.5 / 5.5 and 6.7 / 5.1; 8 MB in one tensor 6.0 / 5.5.  Of more chunks the pieces cost more than they save (62 MB in one tensor
// 20.5 / 20.7 and 20.1 / 22.3): whole, four units per thread in the general path too, the last chunks end sooner (the views
// of perf/cases.py 61.3 / 58.9 and 66.2 / 64.5, 32 MB in tensors of 65 000 bytes 15.1 / 12.8 and 14.1 / 13.1), and so are views of
// several dimensions (62 MB in runs of 1 KiB, a unit after the other 34.4 / 33.3, so 30.6 / 31.1).  In the gather without wide
// blocks that takes 76 registers and leaves six work-groups per CU instead of seven.
// RESTS: chunks that hold little besides blocks (mostly_rests) are moved whole, the general path's units one per thread: there
// is nothing for more.  In pieces or with four units / so: 500 transposed bf16 of 100 x 102 7.7 / 6.1 and 8.2 / 6.7, 1000 of them 10.4 / 9.4
// and 11.2 / 10.5, 3000 25.9 / 23.6 and 36.0 / 34.0, beside as many vectors of 1000 bytes 8.5 / 6.7 and 8.9 / 7.7, 500, 27.8 / 25.6 and
// 38.9 / 37.4, 3000; 500 of every second of 9146 fp32 15.5 / 13.8 and 16.2 / 14.4.
enum : int { kPieces, kWhole, kRests };
template <bool PACK, bool NTL, int HOW, bool WIDE>
__global__ __launch_bounds__(256, 5) void ds_mixed_kernel(const DsPerm *perms, const DsPermItem *items, uint32_t n_items,
                                                          uint32_t xcd_span, uint32_t stripe, uint32_t magic, const DsChunkRec *recs,
                                                          const uint32_t *ids, uint32_t n, uint32_t span, uint32_t c_lo, MoveArgs ma) {
  const PermArgs a = {perms, items, n_items, xcd_span, stripe, magic};
  __shared__ union {
    __attribute__((aligned(16))) uint8_t block[WIDE ? kPermLdsBytes : kPermNarrowBytes];
    GenLds tab;
  } s;
  constexpr int UNITS = HOW == kPieces ? 1 : 4;                      // per thread
  constexpr uint32_t kPerChunk = HOW == kPieces ? kUnitPieces : 1u;  // work-groups
  uint32_t wi = blockIdx.x;
  if (wi < a.xcd_span * 8u) {
    const uint32_t i = ds_perm_ordered(wi, a.stripe, a.magic);
    if (i < a.n_items) move_perm_item<PACK, NTL>(a, ImageArgs{ma.img, ma.img_lo, ma.img_hi}, i, s.block);
    return;
  }
  wi -= a.xcd_span * 8u;
  uint64_t c;
  uint32_t t0, t1, piece;
  if (wi < span * 8u) {
    const uint32_t cm = (wi & 7u) * span + (wi >> 3), rec = c_lo + cm / kPerChunk;
    if (cm >= n) return;
    piece = cm % kPerChunk * 4096;
    const DsChunkRec r = load_rec(recs, rec);
    c = load_id(ids, rec);
    uint8_t *const img = ma.img + ((c << 14) - ma.img_lo);
    if ((r.kind & 0xFFu) < DS_CHUNK_GENERAL) {
      lean_move<PACK, 256, UNITS, NTL, true, PACK>(r, img + piece, piece);
      return;
    }
    if ((r.kind & 0xFFu) == DS_CHUNK_DIMS) {
      dims_move<PACK, 256, UNITS, NTL, PACK>(r, ma.tiles, img + piece, piece);
      return;
    }
    t0 = r.tile;
    t1 = r.tile + r.col0;
  } else {
    const uint32_t x = wi - span * 8u;
    c = ma.extra[x / kPerChunk];
    piece = x % kPerChunk * 4096;
    cut_chunk_tiles(ma, c, t0, t1);
  }
  general_chunk<PACK, 256, HOW == kWhole ? 4 : 1, NTL, true, PACK, kListed, HOW != kPieces>(ma, c, piece, t0, t1, &s.tab);
}

template <bool PACK, bool NTL, int HOW>
int launch_mixed(const ds_plan *plan, const PermArgs &a, const LeanArgs &la, const MoveArgs &ma, hipStream_t stream) {
  constexpr uint32_t kPerChunk = HOW == kPieces ? kUnitPieces : 1u;
  const uint32_t n = la.n_pieces * kPerChunk, span = (n + 7) / 8;
  const dim3 grid(a.xcd_span * 8 + span * 8 + ma.n_extra * kPerChunk);
  if (plan->any_wide)
    hipLaunchKernelGGL((ds_mixed_kernel<PACK, NTL, HOW, true>), grid, dim3(256), 0, stream, a.perms, a.items, a.n_items,
                       a.xcd_span, a.stripe, a.magic, la.recs, la.ids, n, span, la.c_lo, ma);
  else
    hipLaunchKernelGGL((ds_mixed_kernel<PACK, NTL, HOW, false>), grid, dim3(256), 0, stream, a.perms, a.items, a.n_items,
                       a.xcd_span, a.stripe, a.magic, la.recs, la.ids, n, span, la.c_lo, ma);
  DS_HIP_TRY(hipGetLastError());
  return DS_OK;
}
template <bool PACK, bool NTL>
int launch_mixed(const ds_plan *plan, const PermArgs &a, const LeanArgs &la, const MoveArgs &ma, hipStream_t stream) {
  const bool in_pieces = la.n_pieces <= kMixedInPieces;
  return plan->mostly_rests(in_pieces) ? launch_mixed<PACK, NTL, kRests>(plan, a, la, ma, stream)
         : in_pieces                   ? launch_mixed<PACK, NTL, kPieces>(plan, a, la, ma, stream)
                                       : launch_mixed<PACK, NTL, kWhole>(plan, a, la, ma, stream);
}

template <bool PACK, bool STREAM>
int launch_perm(const ds_plan *plan, const PermArgs &a, const ImageArgs &image, uint32_t grid_limit, hipStream_t stream) {
  uint32_t grid = a.xcd_span ? a.xcd_span * 8 : a.n_items;
  if (grid_limit && grid > grid_limit) grid = grid_limit;
  if (grid > kMaxGrid) grid = kMaxGrid;
  if (plan->any_wide) hipLaunchKernelGGL((ds_perm_kernel<PACK, STREAM, true>), dim3(grid), dim3(256), 0, stream, a.perms, a.items,
                                          a.n_items, a.xcd_span, a.stripe, a.magic, image);
  else hipLaunchKernelGGL((ds_perm_kernel<PACK, STREAM, false>), dim3(grid), dim3(256), 0, stream, a.perms, a.items, a.n_items,
                          a.xcd_span, a.stripe, a.magic, image);
  DS_HIP_TRY(hipGetLastError());
  return DS_OK;
}

// A plain contiguous copy in ds_move_kernel's shape (256 threads x 4 units per
// work-group, four wavefronts per SIMD, non-temporal 16-byte accesses): the rate
// the gather is compared with, and the known-size kernel the HBM counters are
// scaled by.  No ceiling: one unit per thread at eight wavefronts, as in
// ds_unit_kernel, copies at 6.75 TB/s, this one at 6.34 to 6.48.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 4))) void ds_copy_probe_kernel(const u32x4 *__restrict__ src, u32x4 *__restrict__ dst,
                                                            uint64_t n_units) {
  // the same XCD-contiguous order of work-groups as the lean path
  const uint32_t n_groups = (uint32_t)((n_units + 1023) / 1024), span = (n_groups + 7) / 8;
  const uint32_t g = (blockIdx.x & 7u) * span + (blockIdx.x >> 3);
  if (g >= n_groups) return;
  const uint64_t first = (uint64_t)g * 1024;  // this work-group's 1024 units
  const uint64_t left = n_units - first;
  const uint32_t mine = left < 1024 ? (uint32_t)left : 1024u;
  __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(dst + first, 0, (int)(mine * 16u), 0x00020000);
  u32x4 v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (threadIdx.x + 256u * i < mine) v[i] = __builtin_nontemporal_load(src + first + threadIdx.x + 256 * i);
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (threadIdx.x + 256u * i < mine)
      __builtin_amdgcn_raw_buffer_store_b128(v[i], out, (int)(16u * (threadIdx.x + 256u * i)), 0, kStorePolicySc0Sc1Nt);
}

// ---- which blocks of two images differ ----------------------------------------------------------
__global__ __launch_bounds__(256) void ds_clear_flags_kernel(uint32_t *flags, uint64_t n) {
  const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) flags[i] = 0;
}

// One work-group compares 1024 units (16 KiB) of the two images, in the lean path's shape and order; a
// wavefront that saw a difference sets the flag of the block its units belong to (a 16 KiB piece never
// straddles two blocks: the block size is a multiple of 16 KiB).
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 4))) void ds_diff_kernel(
    const u32x4 *__restrict__ a, const u32x4 *__restrict__ b, uint64_t n_units, uint32_t units_per_block_log2,
    uint32_t *__restrict__ flags) {
  const uint32_t n_groups = (uint32_t)((n_units + 1023) / 1024), span = (n_groups + 7) / 8;
  const uint32_t g = (blockIdx.x & 7u) * span + (blockIdx.x >> 3);
  if (g >= n_groups) return;
  const uint64_t first = (uint64_t)g * 1024;
  const uint64_t left = n_units - first;
  const uint32_t mine = left < 1024 ? (uint32_t)left : 1024u;
  u32x4 x[4], y[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (threadIdx.x + 256u * i < mine) {
      x[i] = __builtin_nontemporal_load(a + first + threadIdx.x + 256 * i);
      y[i] = __builtin_nontemporal_load(b + first + threadIdx.x + 256 * i);
    }
  uint32_t diff = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (threadIdx.x + 256u * i < mine) {
      const u32x4 d = x[i] ^ y[i];
      diff |= d.x | d.y | d.z | d.w;
    }
  if (__ballot(diff != 0) != 0 && (threadIdx.x & (kWave - 1)) == 0) atomicOr(flags + (first >> units_per_block_log2), 1u);
}

// ---- block elision of an image (the compressed-snapshot experiment) ------------------------------------
// Bound by HBM: the kept blocks are read and written once, the constant ones read once.  A block that is kept
// usually shows it in its first 4 KiB, so the flags cost little more than the constant blocks' bytes and the image
// is read once in all, not twice.  1 GiB of which 30 % is constant, in blocks of 64 KiB: flags, scan and dense
// copy together 603 us with every byte read by both passes (275 + 280 us) and a scan of 256 entries at a time
// (46 us).  Small images are bound by the launches: see ds_count_and_pack_kernel.
//
// One work-group looks at one segment: a whole block of up to 64 KiB, or 64 KiB of a larger one (WHOLE = false; the
// flags are cleared before).  keep[k] = 1 if some 16-byte unit of block k differs from the block's first unit.
template <bool WHOLE>
__global__ __launch_bounds__(256) void ds_constant_segments_kernel(const u32x4 *__restrict__ img, uint64_t n_units,
                                                                   uint32_t units_per_block_log2,
                                                                   uint32_t units_per_segment_log2,
                                                                   uint32_t *__restrict__ keep, u32x4 *__restrict__ patterns) {
  const uint32_t segments = (uint32_t)((n_units + (1ull << units_per_segment_log2) - 1) >> units_per_segment_log2);
  // Work-group i takes segment i, round-robin over the XCDs: constant blocks come in long runs, which in the lean
  // path's order would be the work of one or two of them (99 us instead of 61, with 22 % of the image in one run).
  const uint32_t g = blockIdx.x, tid = threadIdx.x;
  if (g >= segments) return;
  const uint64_t first = (uint64_t)g << units_per_segment_log2, left = n_units - first;
  const uint32_t n = left < (1ull << units_per_segment_log2) ? (uint32_t)left : 1u << units_per_segment_log2;
  const auto [block, in_block] = ds_block_place(first, units_per_block_log2);
  const u32x4 ref = img[first - in_block];
  u32x4 x = ref;
  if (tid < n) x = __builtin_nontemporal_load(img + first + tid);
  u32x4 d = x ^ ref;
  int any = __syncthreads_or((d.x | d.y | d.z | d.w) != 0);
  for (uint32_t base = 256; base < n && !any; base += 1024) {
    u32x4 y[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t u = base + 256u * i + tid;
      y[i] = __builtin_nontemporal_load(img + first + (u < n ? u : n - 1));
    }
    uint32_t diff = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      d = y[i] ^ ref;
      diff |= d.x | d.y | d.z | d.w;
    }
    any = __syncthreads_or(diff != 0);
  }
  if (tid == 0) {
    if (WHOLE) keep[block] = any ? 1u : 0u;
    else if (any) atomicOr(keep + block, 1u);
    if (in_block == 0) patterns[block] = ref;
  }
}

// The same for blocks of 128 KiB to 1 MiB in images of up to 16 MiB: one work-group looks at a block of up to 256 KiB, four at a
// larger one, so that no flags have to be cleared by a launch of their own.  Behind its first 16 KiB a work-group takes the rest
// at once.  Bound by the latency of that where blocks are constant: one CU reads a constant block of 1 MiB in 20 us.
// Four leave a byte of the block's flag each; ds_count_and_pack_kernel makes 1 of them.  All of ds_image_compress, us, one
// work-group per block / in segments / now: 8 MB that no cache holds, all of it constant, in blocks of 128 KiB 8.2 / 11.5, of
// 256 KiB 9.4 / 11.6, of 512 KiB 14.3 / 11.5 / 8.0, of 1 MiB 23.9 / 11.4 / 9.2; in the caches and in a captured graph 6.8 / 9.3,
// 6.4 / 9.5, 8.5 / 9.4 / 6.2, 12.8 / 9.4 / 6.0; nothing constant 5.5 / 7.0, 5.4 / 7.1, 5.2 / 7.6 / 5.5, 5.2 / 7.5 / 5.3.
constexpr uint32_t kBlockThreads = 1024, kBlockUnroll = 16;
template <uint32_t PARTS_LOG2>
__global__ __launch_bounds__(kBlockThreads) void ds_constant_blocks_kernel(const u32x4 *__restrict__ img, uint64_t n_units,
                                                                           uint32_t units_per_block_log2,
                                                                           uint32_t *__restrict__ keep,
                                                                           u32x4 *__restrict__ patterns) {
  const uint32_t tid = threadIdx.x, block = blockIdx.x >> PARTS_LOG2, part = blockIdx.x & ((1u << PARTS_LOG2) - 1);
  const uint32_t units_log2 = units_per_block_log2 - PARTS_LOG2;  // of a work-group
  const uint64_t first = (uint64_t)blockIdx.x << units_log2, left = first < n_units ? n_units - first : 0;
  const uint32_t n = left < (1ull << units_log2) ? (uint32_t)left : 1u << units_log2;  // (0: behind the end of the image)
  const u32x4 ref = img[(uint64_t)block << units_per_block_log2];
  u32x4 d = u32x4{0, 0, 0, 0};
  if (tid < n) d = img[first + tid] ^ ref;
  int any = __syncthreads_or((d.x | d.y | d.z | d.w) != 0);
  for (uint32_t base = kBlockThreads; base < n && !any; base += kBlockUnroll * kBlockThreads) {
    u32x4 y[kBlockUnroll];
#pragma unroll
    for (uint32_t i = 0; i < kBlockUnroll; ++i) {
      const uint32_t u = base + kBlockThreads * i + tid;
      y[i] = img[first + (u < n ? u : n - 1)];
    }
    uint32_t diff = 0;
#pragma unroll
    for (uint32_t i = 0; i < kBlockUnroll; ++i) {
      d = y[i] ^ ref;
      diff |= d.x | d.y | d.z | d.w;
    }
    any = __syncthreads_or(diff != 0);
  }
  if (tid == 0) {
    if (PARTS_LOG2) ((uint8_t *)keep)[blockIdx.x] = any ? 1 : 0;
    else keep[block] = any ? 1u : 0u;
    if (part == 0) patterns[block] = ref;
  }
}

// pos[k] = keep[0] + ... + keep[k-1], pos[n] = the sum.  One work-group walks the array 16 Ki entries at a time, a
// wavefront 1024 neighbouring ones: at that width one step covers a 1 GiB image of 64 KiB blocks (7 us; 16 entries
// per thread one behind the other, each load of a wavefront on 64 lines, 17 us).
constexpr uint32_t kScanThreads = 1024, kScanQuads = 4;  // quads of entries per thread and step
__global__ __launch_bounds__(kScanThreads) void ds_exclusive_scan_kernel(const uint32_t *__restrict__ keep,
                                                                         uint32_t *__restrict__ pos, uint64_t n) {
  __shared__ uint32_t wave_sum[kScanThreads / kWave];
  const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
  uint32_t carry = 0;
  for (uint64_t base = 0; base < n; base += kScanThreads * kScanQuads * 4) {
    const uint64_t at = base + (uint64_t)wv * (kWave * kScanQuads * 4) + lane * 4;
    u32x4 x[kScanQuads];
#pragma unroll
    for (uint32_t j = 0; j < kScanQuads; ++j) {
      const uint64_t i = at + j * (kWave * 4);
      x[j] = u32x4{0, 0, 0, 0};
      if (i + 4 <= n) x[j] = ld16_any<false>((const uint8_t *)(keep + i));
      else
        for (uint32_t e = 0; e < 3; ++e)
          if (i + e < n) x[j][e] = keep[i + e];
    }
    uint32_t before[kScanQuads], sum = 0;  // of the wavefront's entries, those before the quad
#pragma unroll
    for (uint32_t j = 0; j < kScanQuads; ++j) {
      const uint32_t mine = x[j].x + x[j].y + x[j].z + x[j].w;
      const uint32_t incl = wave_inclusive_scan(mine);
      before[j] = sum + incl - mine;
      sum += __shfl(incl, kWave - 1, kWave);
    }
    if (lane == 0) wave_sum[wv] = sum;
    __syncthreads();
    const uint32_t other = lane < kScanThreads / kWave ? wave_sum[lane] : 0u;
    const uint32_t waves = wave_inclusive_scan(other);
    const uint32_t start = carry + __shfl(waves - other, wv, kWave);
    carry += __shfl(waves, kWave - 1, kWave);
#pragma unroll
    for (uint32_t j = 0; j < kScanQuads; ++j) {
      const uint64_t i = at + j * (kWave * 4);
      u32x4 v;
      v.x = start + before[j];
      v.y = v.x + x[j].x;
      v.z = v.y + x[j].y;
      v.w = v.z + x[j].z;
      if (i + 4 <= n) st16_any<false>((uint8_t *)(pos + i), v);
      else
        for (uint32_t e = 0; e < 3; ++e)
          if (i + e < n) pos[i + e] = v[e];
    }
    __syncthreads();
  }
  if (tid == 0) pos[n] = carry;
}

// Kept blocks go to their slots in `packed`, one behind the other.  One work-group takes 256 x UNROLL units (4 or 16
// KiB), which lie in one block (the block size is a power of two of at least 16 KiB).
// Bound by HBM.  One unit per thread at eight wavefronts per SIMD, as in ds_unit_kernel (1 GiB of which 30 % is constant,
// all of ds_image_compress: 305.6 us with four units at four wavefronts, now 299.3); launches of that shape have room for
// images of up to 64 GiB, larger ones take four units per thread.
constexpr uint32_t kStripeUnitsLog2 = 16;
// (A structure, so that the arguments are not in registers from the start: work-groups of constant blocks are many, and
// setting up 12 more scalar registers for each wavefront costs 2 of the 297 us.)
struct KeptArgs {
  const u32x4 *img;
  uint64_t n_units;
  uint32_t units_per_block_log2;
  const uint32_t *keep, *pos;
  u32x4 *packed;
};
template <int UNROLL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 8))) void ds_pack_kept_blocks_kernel(KeptArgs args) {
  const u32x4 *__restrict__ const img = args.img;
  const uint32_t *__restrict__ const keep = args.keep, *__restrict__ const pos = args.pos;
  u32x4 *__restrict__ const packed = args.packed;
  const uint64_t n_units = args.n_units;
  const uint32_t units_per_block_log2 = args.units_per_block_log2;
  constexpr uint32_t kUnits = 256 * UNROLL, kGroupsLog2 = kStripeUnitsLog2 - __builtin_ctz(kUnits);
  // an XCD takes every eighth stripe of 1 MiB: neighbours share an L2, and runs of constant blocks, which leave
  // nothing to do, are dealt evenly (four units per thread 241 us; one contiguous eighth per XCD 271 us)
  const uint32_t i8 = blockIdx.x >> 3;
  const uint32_t g = ((i8 >> kGroupsLog2) * 8 + (blockIdx.x & 7u)) << kGroupsLog2 | (i8 & ((1u << kGroupsLog2) - 1));
  const uint64_t first = (uint64_t)g * kUnits;
  if (first >= n_units) return;
  const uint64_t left = n_units - first;
  const uint32_t mine = left < kUnits ? (uint32_t)left : kUnits;
  const auto [block, in_block] = ds_block_place(first, units_per_block_log2);
  const uint32_t slot = pos[block];
  if (!keep[block]) return;
  u32x4 x[UNROLL];
#pragma unroll
  for (int i = 0; i < UNROLL; ++i)
    if (threadIdx.x + 256u * i < mine) x[i] = __builtin_nontemporal_load(img + first + threadIdx.x + 256 * i);
  __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(packed + ((uint64_t)slot << units_per_block_log2) + in_block,
                                                                 0, (int)(mine * 16u), 0x00020000);
#pragma unroll
  for (int i = 0; i < UNROLL; ++i)
    if (threadIdx.x + 256u * i < mine)
      __builtin_amdgcn_raw_buffer_store_b128(x[i], out, (int)(16u * (threadIdx.x + 256u * i)), 0, kStorePolicySc0Sc1Nt);
}

template <int UNROLL>
int launch_pack_kept(const u32x4 *img, uint64_t n_units, uint32_t upb_log2, const uint32_t *keep, const uint32_t *pos,
                     u32x4 *packed, hipStream_t stream) {
  const uint64_t stripes = ((n_units + (1u << kStripeUnitsLog2) - 1) >> kStripeUnitsLog2);
  const uint32_t grid = (uint32_t)((stripes + 7) / 8 * 8 << (kStripeUnitsLog2 - __builtin_ctz(256 * UNROLL)));
  hipLaunchKernelGGL(ds_pack_kept_blocks_kernel<UNROLL>, dim3(grid), dim3(256), 0, stream,
                     KeptArgs{img, n_units, upb_log2, keep, pos, packed});
  DS_HIP_TRY(hipGetLastError());
  return DS_OK;
}

// The scan and the pack in one launch, for images of up to 64 MiB in up to 2048 blocks: a work-group counts the kept blocks
// in front of its own, whose flags are at most 8 KiB in the L2, and the first of each block leaves the count in pos.
// Small images are bound by the launches, each about 4 us of the caller's time, then by the chain flags -> count -> stores
// behind the loads; from 8 MiB on by the caches and HBM, where four units per thread and ordinary loads are ahead.  All of
// ds_image_compress with the scan of its own / so, us: 16 KB 10.2 / 6.0, 1 MB 10.1 / 6.1, 8 MB in blocks of 256 KiB 13.7 / 6.2 (no
// clearing launch either), 17 MB of which 30 % is constant 16.7 / 13.2 (one unit per thread 13.8), 34 MB in 2048 blocks 18.5 /
// 14.1, 64 MB 27.7 / 25.8, none of it constant 32.9 / 21.9 (streaming loads 27.7).  Beyond: 134 MB in 2048 blocks 45.1 / 42.2,
// none constant 49.5 / 51.7; 256 MB 78.3 / 82.5; 1 GiB in 1024 blocks 307 / 331.
// Those are images that the last-level cache holds from the pass before.  Out of a rotation of 700 MB, blocks of 32 KiB, with
// the scan / so / so with streaming loads: 16 MB 13.4 / 10.6 / 10.3, 34 MB 20.5 / 18.7 / 19.0, 64 MB 30.2 / 30.3 / 30.8; of
// which 30 % is constant 15.0 / 12.4 / 11.7, 19.6 / 17.6 / 17.7, 27.7 / 26.5 / 25.9.
// PARTS: of each block's flag four work-groups left a byte.  These are at most 32 blocks; a wavefront reads all the flags, and the
// first work-group of a block leaves 1 in place of its bytes.  Others may still read them: whole words on either side,
// neither of them 0.  (Such loads pass the caches by: four units per thread from 6 MiB on, 8 MB in blocks of 512 KiB, nothing
// constant, 7.0 / 5.6; 6 MB, half of it constant, one 6.8, four 7.6.)
constexpr uint64_t kCountedBlocks = 2048, kOneUnitBytes = 8ull << 20, kOneUnitPartsBytes = 6ull << 20;
static_assert((kWholeBlocksBytes >> (4 + kOnePartUnitsLog2 + 1)) <= kWave, "a lane per block in parts");
template <int UNROLL, bool PARTS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 8))) void ds_count_and_pack_kernel(
    const u32x4 *__restrict__ img, uint32_t n_units, uint32_t units_per_block_log2, uint32_t *keep, uint32_t *__restrict__ pos,
    uint32_t n_blocks, u32x4 *__restrict__ packed) {
  __shared__ uint32_t wave_sum[256 / kWave];
  constexpr uint32_t kUnits = 256 * UNROLL;  // in one block (of a power of two of at least 16 KiB)
  const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1);
  const uint32_t first = blockIdx.x * kUnits, left = n_units - first, mine = left < kUnits ? left : kUnits;
  const DsBlockPlace place = ds_block_place(first, units_per_block_log2);
  const uint32_t block = (uint32_t)place.block, in_block = (uint32_t)place.in_block;  // less than 2048, and 2^22
  uint64_t flags = 0;
  if (PARTS) {
    uint32_t flag = 0;
    if (lane < n_blocks) flag = __hip_atomic_load(keep + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    flags = __ballot(flag != 0);
  }
  const uint32_t kept = PARTS ? (uint32_t)(flags >> block) & 1u : keep[block];
  if (!kept && in_block) return;
  u32x4 x[UNROLL];
  if (kept) {
#pragma unroll
    for (uint32_t i = 0; i < UNROLL; ++i)
      if (tid + 256u * i < mine) x[i] = img[first + tid + 256u * i];
  }
  uint32_t slot = 0;
  if (PARTS) {
    slot = (uint32_t)__popcll(flags & ((1ull << block) - 1));
    if (tid == 0 && in_block == 0 && kept) __hip_atomic_store(keep + block, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else {
    uint32_t sum = 0;
    for (uint32_t i = tid * 4; i < block; i += 1024) {
      u32x4 v = u32x4{0, 0, 0, 0};
      if (i + 4 <= n_blocks) v = ld16_any<false>((const uint8_t *)(keep + i));
      else
        for (uint32_t e = 0; e < 3; ++e)
          if (i + e < n_blocks) v[e] = keep[i + e];
      sum += v.x + (i + 1 < block ? v.y : 0u) + (i + 2 < block ? v.z : 0u) + (i + 3 < block ? v.w : 0u);
    }
    sum = wave_inclusive_scan(sum);
    if (lane == kWave - 1) wave_sum[tid / kWave] = sum;
    __syncthreads();
    slot = wave_sum[0] + wave_sum[1] + wave_sum[2] + wave_sum[3];
  }
  if (tid == 0 && in_block == 0) {
    pos[block] = slot;
    if (block + 1 == n_blocks) pos[n_blocks] = slot + kept;
  }
  if (!kept) return;
  __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(packed + ((uint64_t)slot << units_per_block_log2) + in_block,
                                                                 0, (int)(mine * 16u), 0x00020000);
#pragma unroll
  for (uint32_t i = 0; i < UNROLL; ++i)
    if (tid + 256u * i < mine)
      __builtin_amdgcn_raw_buffer_store_b128(x[i], out, (int)(16u * (tid + 256u * i)), 0, kStorePolicySc0Sc1Nt);
}

}  // namespace

extern "C" int ds_image_compress(const void *image_dev, uint64_t nbytes, uint64_t block_bytes, uint32_t *keep_dev,
                                 uint32_t *pos_dev, void *patterns_dev, void *packed_dev, void *stream) {
  if (nbytes == 0) return DS_OK;
  if (!image_dev || !keep_dev || !pos_dev || !patterns_dev || !packed_dev ||
      (((uintptr_t)image_dev | (uintptr_t)patterns_dev | (uintptr_t)packed_dev) & 15) ||
      (((uintptr_t)keep_dev | (uintptr_t)pos_dev) & 3))
    return DS_EINVAL;
  // a power of two of at least 16 KiB, so that a work-group's piece lies in one block
  if (block_bytes < 16384 || (block_bytes & (block_bytes - 1)) || (nbytes & 15)) return DS_ERANGE;
  const uint64_t n_units = nbytes >> 4;
  const uint64_t groups = (n_units + 1023) / 1024;
  if (groups > 0x7FFFFFF0ull) return DS_ERANGE;
  const uint64_t n_blocks = (nbytes + block_bytes - 1) / block_bytes;
  const uint32_t upb_log2 = (uint32_t)__builtin_ctzll(block_bytes >> 4);
  hipStream_t st = (hipStream_t)stream;
  const uint32_t ups_log2 = upb_log2 < kSegmentUnitsLog2 ? upb_log2 : kSegmentUnitsLog2;
  const uint64_t segments = (n_units + (1ull << ups_log2) - 1) >> ups_log2;
  const dim3 seg_grid((uint32_t)segments);
  const int parts_log2 = ds_block_parts_log2(nbytes, upb_log2);
  if (parts_log2 == 0) {
    hipLaunchKernelGGL(ds_constant_blocks_kernel<0>, dim3((uint32_t)n_blocks), dim3(kBlockThreads), 0, st,
                       (const u32x4 *)image_dev, n_units, upb_log2, keep_dev, (u32x4 *)patterns_dev);
  } else if (parts_log2 > 0) {
    hipLaunchKernelGGL(ds_constant_blocks_kernel<kBlockPartsLog2>, dim3((uint32_t)n_blocks << kBlockPartsLog2), dim3(kBlockThreads), 0,
                       st, (const u32x4 *)image_dev, n_units, upb_log2, keep_dev, (u32x4 *)patterns_dev);
  } else if (ups_log2 == upb_log2) {
    hipLaunchKernelGGL(ds_constant_segments_kernel<true>, seg_grid, dim3(256), 0, st, (const u32x4 *)image_dev, n_units,
                       upb_log2, ups_log2, keep_dev, (u32x4 *)patterns_dev);
  } else {
    hipLaunchKernelGGL(ds_clear_flags_kernel, dim3((uint32_t)((n_blocks + 255) / 256)), dim3(256), 0, st, keep_dev, n_blocks);
    DS_HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(ds_constant_segments_kernel<false>, seg_grid, dim3(256), 0, st, (const u32x4 *)image_dev, n_units,
                       upb_log2, ups_log2, keep_dev, (u32x4 *)patterns_dev);
  }
  DS_HIP_TRY(hipGetLastError());
  if (n_blocks <= kCountedBlocks && nbytes <= kCachedBytes) {
    const auto launch = [&](auto kernel, uint32_t units) {
      hipLaunchKernelGGL(kernel, dim3((uint32_t)((n_units + units - 1) / units)), dim3(256), 0, st, (const u32x4 *)image_dev,
                         (uint32_t)n_units, upb_log2, keep_dev, pos_dev, (uint32_t)n_blocks, (u32x4 *)packed_dev);
    };
    const bool parts = parts_log2 > 0;
    if (nbytes <= (parts ? kOneUnitPartsBytes : kOneUnitBytes)) launch(parts ? ds_count_and_pack_kernel<1, true> : ds_count_and_pack_kernel<1, false>, 256);
    else launch(parts ? ds_count_and_pack_kernel<4, true> : ds_count_and_pack_kernel<4, false>, 1024);
    DS_HIP_TRY(hipGetLastError());
    return DS_OK;
  }
  hipLaunchKernelGGL(ds_exclusive_scan_kernel, dim3(1), dim3(kScanThreads), 0, st, keep_dev, pos_dev, n_blocks);
  DS_HIP_TRY(hipGetLastError());
  // (launches have less than 2^32 threads, and are rounded up to 8 MiB of image)
  return n_units <= (1ull << 32) - (16u << kStripeUnitsLog2)
             ? launch_pack_kept<1>((const u32x4 *)image_dev, n_units, upb_log2, keep_dev, pos_dev, (u32x4 *)packed_dev, st)
             : launch_pack_kept<4>((const u32x4 *)image_dev, n_units, upb_log2, keep_dev, pos_dev, (u32x4 *)packed_dev, st);
}

extern "C" int ds_image_diff(const void *image_a_dev, const void *image_b_dev, uint64_t nbytes, uint64_t block_bytes,
                             uint32_t *changed_dev, void *stream) {
  if (nbytes == 0) return DS_OK;
  if (!image_a_dev || !image_b_dev || !changed_dev || (((uintptr_t)image_a_dev | (uintptr_t)image_b_dev) & 15) ||
      ((uintptr_t)changed_dev & 3))
    return DS_EINVAL;
  // a power of two of at least 16 KiB, so that a work-group's piece lies in one block
  if (block_bytes < 16384 || (block_bytes & (block_bytes - 1)) || (nbytes & 15)) return DS_ERANGE;
  const uint64_t n_units = nbytes >> 4;
  const uint64_t groups = (n_units + 1023) / 1024;
  if (groups > 0x7FFFFFF0ull) return DS_ERANGE;
  const uint64_t n_blocks = (nbytes + block_bytes - 1) / block_bytes;
  hipLaunchKernelGGL(ds_clear_flags_kernel, dim3((uint32_t)((n_blocks + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                     changed_dev, n_blocks);
  DS_HIP_TRY(hipGetLastError());
  const uint64_t grid = ((groups + 7) / 8) * 8;
  hipLaunchKernelGGL(ds_diff_kernel, dim3((uint32_t)grid), dim3(256), 0, (hipStream_t)stream, (const u32x4 *)image_a_dev,
                     (const u32x4 *)image_b_dev, n_units, (uint32_t)__builtin_ctzll(block_bytes >> 4), changed_dev);
  DS_HIP_TRY(hipGetLastError());
  return DS_OK;
}

extern "C" int ds_copy_probe(void *dst_dev, const void *src_dev, uint64_t nbytes, void *stream) {
  if (nbytes == 0) return DS_OK;
  if (!dst_dev || !src_dev || (((uintptr_t)dst_dev | (uintptr_t)src_dev | nbytes) & 15)) return DS_EINVAL;
  const uint64_t n_units = nbytes >> 4;
  const uint64_t groups = (n_units + 1023) / 1024;
  if (groups > 0x7FFFFFF0ull) return DS_ERANGE;
  const uint64_t grid = ((groups + 7) / 8) * 8;
  hipLaunchKernelGGL(ds_copy_probe_kernel, dim3((uint32_t)grid), dim3(256), 0, (hipStream_t)stream,
                     (const u32x4 *)src_dev, (u32x4 *)dst_dev, n_units);
  DS_HIP_TRY(hipGetLastError());
  return DS_OK;
}

namespace {

// The plan's tables in device memory: the plan's own copy, or the one ds_pack_noalloc keeps in static memory.
struct DeviceTables {
  const DsTile *tiles;
  const DsTileHot *hot;
  const uint32_t *first_tile;
  const DsChunkRec *recs;
  const DsPerm *perms;             // null: no block tables, the general path takes those views
  const DsPermItem *perm_items;
  const uint32_t *rest_ids;        // plan->listed: the chunks left beside them
  const DsChunkRec *rest_recs;
};

// What the launch of the range's chunks, lean and general, takes.
void chunk_args(const ds_plan *plan, const DeviceTables &tb, uint8_t *img, uint64_t img_lo, uint64_t img_hi, LeanArgs &la,
                MoveArgs &ma) {
  const uint32_t lg = plan->chunk_log2;
  const uint64_t C = (uint64_t)1 << lg;
  const uint64_t n_total = plan->n_chunks();
  // whole chunks inside the range: one work item each, lean or general by their record ...
  uint64_t w_lo = (img_lo + C - 1) >> lg;
  uint64_t w_hi = img_hi >> lg;
  if (img_hi == plan->total_bytes) w_hi = n_total;  // the last chunk may be short; its record says 'general' then
  la.recs = tb.recs;
  la.ids = nullptr;
  la.img = img;
  la.img_lo = img_lo;
  la.chunk_log2 = lg;
  la.c_lo = (uint32_t)w_lo;
  la.n_pieces = w_hi > w_lo ? (uint32_t)(w_hi - w_lo) : 0;
  if (tb.perms && plan->listed && la.n_pieces) {
    const auto first = std::lower_bound(plan->rest_ids.begin(), plan->rest_ids.end(), (uint32_t)w_lo);
    const auto last = std::lower_bound(first, plan->rest_ids.end(), (uint32_t)w_hi);
    la.recs = tb.rest_recs;
    la.ids = tb.rest_ids;
    la.c_lo = (uint32_t)(first - plan->rest_ids.begin());
    la.n_pieces = (uint32_t)(last - first);
  }
  la.xcd_span = 0;  // launch_pieces makes pieces of the chunks and orders them
  // ... and the one or two chunks cut by the ends of the range, clipped by the general path
  ma.tiles = tb.tiles;
  ma.hot = tb.hot;
  ma.first_tile = tb.first_tile;
  ma.img = img;
  ma.img_lo = img_lo;
  ma.img_hi = img_hi;
  ma.total = plan->total_bytes;
  ma.chunk_log2 = lg;
  ma.n_extra = 0;
  ma.extra[0] = ma.extra[1] = 0;
  const uint64_t c_first = img_lo >> lg, c_last = (img_hi - 1) >> lg;
  if (w_hi <= w_lo) {
    // no whole chunk: the range touches one or two chunks, both cut
    ma.extra[ma.n_extra++] = (uint32_t)c_first;
    if (c_last != c_first) ma.extra[ma.n_extra++] = (uint32_t)c_last;
  } else {
    if (c_first < w_lo) ma.extra[ma.n_extra++] = (uint32_t)c_first;
    if (c_last >= w_hi) ma.extra[ma.n_extra++] = (uint32_t)c_last;
  }
}

// The chunks of the range in one launch.
int launch_chunks(const ds_plan *plan, const DeviceTables &tb, bool pack, const LeanArgs &la, const MoveArgs &ma,
                  uint32_t grid_limit, hipStream_t stream) {
  const uint32_t lg = plan->chunk_log2;
  const uint64_t variant = ds_cfg_variant();
  const bool few = variant == 5 || grid_limit;
  const bool mostly_general = plan->mostly_general(tb.perms != nullptr) && variant != 5;
  // the default, up to images of 64 GiB (a launch has less than 2^32 threads)
  if ((variant == 0 || variant == 4) && !grid_limit && lg == 14 && la.n_pieces < (1u << 22) - 16 &&
      !(mostly_general && plan->all_contiguous)) {
    const int blocks = !tb.perms ? kAlone : plan->listed ? kListed : kBeside;
    if (variant == 0 && plan->mostly_several(blocks != kAlone))
      return blocks == kAlone    ? launch_several<kAlone>(plan, pack, la, ma, stream)
             : blocks == kListed ? launch_several<kListed>(plan, pack, la, ma, stream)
                                 : launch_several<kBeside>(plan, pack, la, ma, stream);
    if (pack)
      return blocks == kAlone    ? launch_units<true, kAlone>(plan, la, ma, stream)
             : blocks == kListed ? launch_units<true, kListed>(plan, la, ma, stream)
                                 : launch_units<true, kBeside>(plan, la, ma, stream);
    return blocks == kAlone    ? launch_units<false, kAlone>(plan, la, ma, stream)
           : blocks == kListed ? launch_units<false, kListed>(plan, la, ma, stream)
                               : launch_units<false, kBeside>(plan, la, ma, stream);
  }
  if (tb.perms)  // (variants 1, 2 and 5 are given no block tables)
    return plan->listed ? launch_beside_blocks<kListed>(plan, pack, few, mostly_general, la, ma, grid_limit, stream)
                        : launch_beside_blocks<kBeside>(plan, pack, few, mostly_general, la, ma, grid_limit, stream);
  if (variant == 1)  // plain loads and stores
    return pack ? launch_gather<false, false, false>(la, ma, grid_limit, stream)
                : launch_scatter<false, false>(plan, few, mostly_general, la, ma, grid_limit, stream);
  if (variant == 2)  // non-temporal global loads and stores everywhere (no buffer stores)
    return pack ? launch_gather<true, true, false>(la, ma, grid_limit, stream)
                : launch_scatter<true, true>(plan, few, mostly_general, la, ma, grid_limit, stream);
  // default: non-temporal accesses, and the lean gather writes the image with "sc0 sc1 nt" buffer stores
  if (mostly_general && plan->all_contiguous && !grid_limit) {
    if (plan->total_bytes <= kCachedBytes)
      return pack ? launch_gather<false, true, true, 8, kAlone, kMulti>(la, ma, grid_limit, stream)
                  : launch_scatter<false, true, kAlone, kMulti>(plan, few, mostly_general, la, ma, grid_limit, stream);
    return pack ? launch_gather<true, true, true, 8, kAlone, kMulti>(la, ma, grid_limit, stream)
                : launch_scatter<true, true, kAlone, kMulti>(plan, few, mostly_general, la, ma, grid_limit, stream);
  }
  if (!pack) return launch_scatter<true, true>(plan, few, mostly_general, la, ma, grid_limit, stream);
  if (mostly_general) return launch_gather<true, true, true, 6>(la, ma, grid_limit, stream);
  return launch_gather<true, true, true>(la, ma, grid_limit, stream);
}

int launch_move_with(const ds_plan *plan, DeviceTables tb, bool pack, uint8_t *img, uint64_t img_lo, uint64_t img_hi,
                     uint32_t grid_limit, hipStream_t stream) {
  const uint64_t variant = ds_cfg_variant();
  if (variant == 1 || variant == 2 || variant == 5) tb.perms = nullptr;
  if (img_hi > plan->total_bytes || img_lo >= img_hi) return DS_ERANGE;
  LeanArgs la;
  MoveArgs ma;
  chunk_args(plan, tb, img, img_lo, img_hi, la, ma);
  if (!tb.perms) return launch_chunks(plan, tb, pack, la, ma, grid_limit, stream);
  // the views that are moved in blocks and have a whole unit in the range; of the first and the last the blocks in it
  const auto v0 = std::upper_bound(plan->perms.begin(), plan->perms.end(), img_lo,
                                   [](uint64_t at, const DsPerm &d) { return at < d.end16; });
  const auto v1 = std::lower_bound(v0, plan->perms.end(), img_hi, [](const DsPerm &d, uint64_t at) { return d.img < at; });
  PermArgs a = {};
  if (v0 != v1) {
    uint64_t first, last, other;
    ds_perm_range(*v0, img_lo, img_hi, &first, &other);
    ds_perm_range(*(v1 - 1), img_lo, img_hi, &other, &last);
    first += plan->perm_first[v0 - plan->perms.begin()];
    last += plan->perm_first[v1 - 1 - plan->perms.begin()];
    a.perms = tb.perms;
    a.items = tb.perm_items + first;
    a.n_items = (uint32_t)(last - first);
    if (variant != 3 && a.n_items < kPermOrdered) {
      const DsPermOrder order = ds_perm_order(a.n_items, pack, pack ? plan->mostly_far() : plan->mostly_columns());
      a.xcd_span = order.span;
      a.stripe = order.stripe;
      a.magic = order.magic;
    }
    if (plan->listed && (variant == 0 || variant == 4) && !grid_limit && plan->chunk_log2 == 14 &&
        la.n_pieces <= kMixedChunks && a.n_items < kMaxGrid / 2) {
      if (plan->total_bytes <= kCachedBytes)
        return pack ? launch_mixed<true, false>(plan, a, la, ma, stream) : launch_mixed<false, false>(plan, a, la, ma, stream);
      return pack ? launch_mixed<true, true>(plan, a, la, ma, stream) : launch_mixed<false, true>(plan, a, la, ma, stream);
    }
  }
  const int rc = launch_chunks(plan, tb, pack, la, ma, grid_limit, stream);
  if (rc != DS_OK || v0 == v1) return rc;
  const ImageArgs image = {img, img_lo, img_hi};
  if (plan->total_bytes <= kCachedBytes)
    return pack ? launch_perm<true, false>(plan, a, image, grid_limit, stream) : launch_perm<false, false>(plan, a, image, grid_limit, stream);
  return pack ? launch_perm<true, true>(plan, a, image, grid_limit, stream) : launch_perm<false, true>(plan, a, image, grid_limit, stream);
}

}  // namespace

int ds_launch_move(const ds_plan *plan, bool pack, uint8_t *img, uint64_t img_lo, uint64_t img_hi,
                   uint32_t grid_limit, hipStream_t stream) {
  // the tables live on the device the plan was made on: a launch from another one would read them remotely
  int dev = -1;
  DS_HIP_TRY(hipGetDevice(&dev));
  if (dev != plan->device) return DS_ESTATE;
  const DeviceTables tb = {plan->d_tiles, plan->d_hot, plan->d_first_tile, plan->d_recs, plan->d_perms,
                           plan->d_perm_items, plan->d_rest_ids, plan->d_rest_recs};
  return launch_move_with(plan, tb, pack, img, img_lo, img_hi, grid_limit, stream);
}

// ---- the gather of few contiguous tensors, whose table travels in the kernel's arguments ---------
// For ds_pack_noalloc, which would copy the plan's tables in front of every launch.  A wavefront's lane i reads tile i (so
// at most 64 of them); the tiles of the wavefront's 64 units are found by two ballots and taken out of the lanes that hold
// them, so the data are one load behind the arguments, as they are one record behind them in ds_unit_kernel.
// Bound by its launch in small images, then by HBM.  The tables copied / in the arguments, us: 24 bf16 tensors of 3 MB 10.1 /
// 7.0 (6.5 is what the caller's loop takes without them), 48 of 25 MB 28.7 / 8.6, 24 of 48 MB 37.6 / 14.5, 48 of 403 MB 162 /
// 128: the copy grows with the image, 36 bytes per 16 KiB, and a kernel behind it starts when it has ended.
namespace {

constexpr uint32_t kArgTiles = 64;
struct ArgTile {
  uint64_t src;
  uint32_t begin;   // image offset in units
  uint32_t nbytes;  // payload
};
struct ArgTiles {
  ArgTile t[kArgTiles];
};

template <bool NTL>
__global__ __launch_bounds__(256) void ds_args_kernel(ArgTiles tiles, uint8_t *img0, uint32_t n_tiles, uint32_t u_lo,
                                                      uint32_t u_hi, uint32_t span) {
  const uint32_t wi = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1);
  const uint64_t at = (uint64_t)u_lo + ((uint64_t)((wi & 7u) * span + (wi >> 3)) << 8);  // the work-group's first unit
  if (at >= u_hi) return;
  const uint32_t first = (uint32_t)at, u = first + tid, w0 = first + (tid - lane);
  ArgTile mine = tiles.t[lane];
  if (lane >= n_tiles) mine.begin = 0xFFFFFFFFu;
  // tile 0 begins with the image: there is one that holds unit w0
  const int t0 = __builtin_popcountll(__ballot(mine.begin <= w0)) - 1;
  const int t1 = __builtin_popcountll(__ballot(mine.begin <= w0 + (kWave - 1))) - 1;
  const auto tile = [&](int k) {
    return ArgTile{(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mine.src, k) |
                       (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(mine.src >> 32), k) << 32,
                   (uint32_t)__builtin_amdgcn_readlane((int)mine.begin, k),
                   (uint32_t)__builtin_amdgcn_readlane((int)mine.nbytes, k)};
  };
  ArgTile t = tile(t0);
  for (int k = t0 + 1; k <= t1; ++k) {
    const ArgTile next = tile(k);
    if (next.begin <= u) t = next;
  }
  const uint64_t d = (uint64_t)(u - t.begin) << 4;
  const uint8_t *p = reinterpret_cast<const uint8_t *>(t.src + d);
  u32x4 v = u32x4{0, 0, 0, 0};
  if (u < u_hi) {
    if (d + 16 <= t.nbytes) v = ld16_aligned<NTL>(p);
    else if (d < t.nbytes) v = load_low_bytes(p, t.nbytes - (uint32_t)d);
  }
  const uint32_t mine_units = u_hi - first < 256 ? u_hi - first : 256u;
  __amdgpu_buffer_rsrc_t out =
      __builtin_amdgcn_make_buffer_rsrc(img0 + ((uint64_t)first << 4), 0, (int)(mine_units * 16), 0x00020000);
  __builtin_amdgcn_raw_buffer_store_b128(v, out, (int)(16 * tid), 0, kStorePolicySc0Sc1Nt);
}

// Up to 64 contiguous tensors of less than 4 GiB each, at multiples of 16 bytes: others have loads that the records
// prepare (DS_CHUNK_REALIGN), or rows.
bool fits_arguments(const ds_plan *plan) {
  if (plan->tiles.size() > kArgTiles || plan->n_strided || plan->total_bytes > (16ull << 30) || ds_cfg_variant()) return false;
  for (const DsTile &t : plan->tiles)
    if (t.nbytes >> 32 || (t.src & 15)) return false;
  return true;
}

int launch_with_arguments(const ds_plan *plan, uint8_t *img, uint64_t img_lo, uint64_t img_hi, hipStream_t stream) {
  ArgTiles tiles = {};
  for (size_t i = 0; i < plan->tiles.size(); ++i)
    tiles.t[i] = ArgTile{plan->tiles[i].src, (uint32_t)(plan->tile_off[i] >> 4), (uint32_t)plan->tiles[i].nbytes};
  const uint32_t u_lo = (uint32_t)(img_lo >> 4), u_hi = (uint32_t)(img_hi >> 4);
  const uint32_t span = ((u_hi - u_lo + 255) / 256 + 7) / 8;
  const dim3 grid(span * 8);
  uint8_t *const img0 = img - img_lo;
  const uint32_t n = (uint32_t)plan->tiles.size();
  if (plan->total_bytes <= kCachedBytes)
    hipLaunchKernelGGL(ds_args_kernel<false>, grid, dim3(256), 0, stream, tiles, img0, n, u_lo, u_hi, span);
  else
    hipLaunchKernelGGL(ds_args_kernel<true>, grid, dim3(256), 0, stream, tiles, img0, n, u_lo, u_hi, span);
  DS_HIP_TRY(hipGetLastError());
  return DS_OK;
}

}  // namespace

// ---- ds_pack for callers that cannot allocate ----------------------------------------------------
// The gather reads the plan's tables from device memory; ds_plan_create puts them into an allocation of
// its own.  Here they go into a static device array instead, so that neither the plan (made with
// DS_PLAN_HOST_ONLY) nor the call allocates device memory.  Every device the library runs on holds its own
// copy of the array, at its own address, until the process ends.
namespace {

constexpr size_t kScratchBytes = DS_PACK_NOALLOC_TABLE_BYTES;
static __device__ __align__(256) uint8_t scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
uint8_t *g_scratch_ptr[kMaxDevices];  // device address of `scratch` on device d, once asked for

// The array's address on the current device (`dev`).  In host code the array's name is only a handle for
// this lookup, never an address a kernel or a copy could use.
int scratch_on_device(int dev, uint8_t **out) {
  if (dev < 0 || dev >= kMaxDevices) return DS_EINVAL;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    DS_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return DS_EINVAL;
    g_scratch_ptr[dev] = (uint8_t *)p;
  }
  *out = g_scratch_ptr[dev];
  return DS_OK;
}

}  // namespace

extern "C" int ds_pack_noalloc(const ds_plan *plan, void *dst_dev, uint64_t img_lo, uint64_t img_hi, void *stream) {
  if (!plan) return DS_EINVAL;
  if (img_lo > img_hi || img_hi > plan->total_bytes || ((img_lo | img_hi) & 15)) return DS_ERANGE;
  if (plan->at.perms > kScratchBytes) return DS_ETOOBIG;  // the tables without those of views moved in blocks
  if (img_lo == img_hi) return DS_OK;
  if (!dst_dev || ((uintptr_t)dst_dev & 15)) return DS_EINVAL;
  if (fits_arguments(plan)) return launch_with_arguments(plan, (uint8_t *)dst_dev, img_lo, img_hi, (hipStream_t)stream);
  int dev = -1;
  DS_HIP_TRY(hipGetDevice(&dev));
  uint8_t *base = nullptr;
  const int rc = scratch_on_device(dev, &base);
  if (rc != DS_OK) return rc;
  // Copy and kernel on the caller's stream: they run behind whatever that stream still has to do with the
  // array (an earlier call's kernel).  Every entry the kernel reads is written here first, so nothing of an
  // earlier call's tables, which stay in the array, needs clearing.  The host tables belong to the plan, which
  // the caller keeps until the work has run.  One copy where the plan holds them so: each is a launch of the runtime's
  // copy kernel (two layers of a small model, 3 MB: 19.0 us with a copy for each of the four tables, 9.4 us with one).
  hipStream_t st = (hipStream_t)stream;
  // the block tables where they fit behind the others; where they do not, the general path takes those views
  const bool blocks = plan->at.total <= kScratchBytes;
  const int copied = ds_copy_tables(plan, blocks, base, st);
  if (copied != DS_OK) return copied;
  DeviceTables tb = {(const DsTile *)base, (const DsTileHot *)(base + plan->at.hot),
                     (const uint32_t *)(base + plan->at.first_tile), (const DsChunkRec *)(base + plan->at.recs),
                     nullptr, nullptr, nullptr, nullptr};
  if (!plan->perms.empty() && blocks) {
    tb.perms = (const DsPerm *)(base + plan->at.perms);
    tb.perm_items = (const DsPermItem *)(base + plan->at.perm_items);
    tb.rest_ids = (const uint32_t *)(base + plan->at.rest_ids);
    tb.rest_recs = (const DsChunkRec *)(base + plan->at.rest_recs);
  }
  return launch_move_with(plan, tb, true, (uint8_t *)dst_dev, img_lo, img_hi, 0, st);
}
