// Views whose contiguous runs are shorter than 16 bytes (transposed and permuted matrices, channels-last
// weights, every k-th column): moved in two-dimensional blocks through LDS instead of unit by unit.
//
// In image order the elements of such a view lie a stride apart, so a 16-byte image unit touches as many
// lines of the tensor as it has elements, and every one of those lines again for the neighbouring rows.  A
// block takes `ta` steps along the dimension whose elements are closest to each other in the TENSOR (a) and
// `tb` steps along the last dimension, whose elements are neighbours in the IMAGE (b); it is read along one
// of them, kept in LDS in image order, and written along the other, so that both sides see whole lines.
//
// What moves is a granule: the largest power of two up to 8 bytes that divides the runs, the strides and the
// base address.
//
// The file compiles for the device and, unchanged, for the host: a CPU test runs the same phases thread by
// thread, with every access checked (DS_PERM_TOUCH).
#pragma once

#include <stdint.h>
#include <string.h>

#include "ds_splice.h"

#if defined(__HIPCC__)
#define DS_PERM_FN __host__ __device__ __forceinline__
#else
#define DS_PERM_FN static inline
#endif
// The plan's tables do not change while a kernel runs: as constant memory they are read into scalar registers, once.
// (Through ordinary pointers, which the stores of a block might change, the compiler reads a field again at every use.)
#if defined(__HIP_DEVICE_COMPILE__)
#define DS_PERM_GLOBAL __attribute__((address_space(1)))
#define DS_PERM_TABLE __attribute__((address_space(4)))
#else
#define DS_PERM_GLOBAL
#define DS_PERM_TABLE
#endif
#ifndef DS_PERM_TOUCH  // the CPU test's hook: (kind, address or LDS offset, bytes, alignment); kind 's': a streaming load
#define DS_PERM_TOUCH(kind, at, n, align)
#endif

constexpr uint32_t kPermThreads = 256;
constexpr uint32_t kPermLdsBytes = 32000;  // five work-groups per CU
constexpr uint32_t kPermNarrowBytes = 21504;  // of which the blocks that are not wide use so many
constexpr uint32_t kPermMaxBatch = 4;      // dimensions beside a and b (DS_MAX_DIMS - 2)
// Smaller views, and views whose blocks would hold less, stay with the general path, which takes 64 tiles at a time.
// Gather of 20 000 square bf16 views, blocks / general path: of 512 bytes 62 / 40 us, of 1152 bytes 69 / 81, of 2048
// bytes 76 / 92, of 4608 bytes 112 / 258; of 2000 views the blocks win from 512 bytes on (10.5 / 25 us).
constexpr uint64_t kPermMinBytes = 1024;
// Images of at most so many bytes have smaller blocks, which all run at once: what one takes is what the launch takes.  (Larger ones
// have more blocks than run at once, and pay for each.)
constexpr uint64_t kPermFewBytes = 2ull << 20;
constexpr uint64_t kPermCacheBytes = 256ull << 20;  // the last-level cache
constexpr int kPermUnroll = 8;             // granules a thread has in flight

enum : uint32_t { kPermAlongA = 1u << 8, kPermFlat = 1u << 9, kPermFull = 1u << 10, kPermLines = 1u << 11,
                  kPermWide = 1u << 12, kPermStream = 1u << 13, kPermOnce = 1u << 14,
                  kPermGroups = 1u << 15, kPermImageOnce = 1u << 16 };

// Wide blocks: views dense along a (16-byte loads of neighbours along a, transposed in registers), kPermWideA steps along a;
// of each row 384 bytes where rows start at lines of the image, else up to 368, and a block writes the lines that start in
// its part of a row.  LDS rows hold 496 bytes: 368 and the 127 up to the end of the last line.
// What bounds a transposition is how much of a line one store has: a plain one of 8192 x 8256 16-bit elements with whole
// lines and streaming stores takes 53 us, with 128 bytes that straddle two lines 69 (cached) or 115 (streaming).  Reading
// up to 127 bytes of a row twice costs less (55 to 57 us).  Gather / scatter, the blocks of before (128 bytes by 256,
// elements one by one through LDS) and these, us: bf16 8192 x 8216 68.5 / 73.9, now 56.1 / 57.8; 8208 x 8232 82.2 / 93.6,
// now 63.6 / 85.6; bytes 48.2 / 54.0, now 28.5 / 47.2; 4096 x 4120 17.6 / 16.4, now 13.5 / 12.5; four transposed 4096 x
// 1024 15.9 / 16.2, now 13.6 / 13.1.  Blocks of 64 x 880 bytes in 64 KB of LDS measure the same.
constexpr uint32_t kPermWideA = 64, kPermWidePitch = 496, kPermWideRow = 368, kPermWideLines = 384, kPermLine = 128;

// Steps along a of the usual block, by granule: at least a 128-byte line of the tensor.
// Its columns are what LDS has room for: a thread's 16 granules (words of up to 4 bytes), all in flight at once.
DS_PERM_FN constexpr uint32_t ds_perm_full_a(uint32_t granule) { return granule == 1 ? 128 : granule == 8 ? 32 : 64; }
DS_PERM_FN constexpr uint32_t ds_perm_full_b(uint32_t granule) { return granule < 4 ? 128 : 64; }

struct DsPerm {
  uint64_t src;    // address of element (0,...,0)
  uint64_t img;    // image offset of the view's first byte
  uint64_t end16;  // image offset where its whole 16-byte units end (the cut unit and padding are the general path's)
  uint64_t sa, sb; // tensor distance between neighbours along a and b, bytes
  uint64_t da;     // image distance between neighbours along a (along b it is `run`)
  uint64_t bsrc[kPermMaxBatch], bimg[kPermMaxBatch];  // the other dimensions, slowest first
  uint32_t bext[kPermMaxBatch];
  uint32_t n_batch;
  uint32_t ea, eb;            // extents
  uint32_t run;               // bytes of a run
  uint32_t ta, tb;            // block size
  uint32_t tiles_a, tiles_b;  // blocks along a and b
  uint32_t pitch;             // LDS bytes between rows of the block
  uint32_t lanes_log2;        // threads that share a row on the image side
  uint32_t flags;             // log2(granule) | kPermAlongA (tensor side walked along a) | kPermFlat | kPermFull (the
                              // usual block) | kPermLines (rows are whole 128-byte lines of the image, or the block
                              // is one piece of it, of which only the two ends are parts of lines) | kPermWide |
                              // kPermStream (wide, and the columns of the tensor start at multiples of 64 bytes: the
                              // scatter's stores stream.  Streaming / cached, us: fp32 4096 x 4099 21.2 / 29.3, bytes
                              // 8192 x 8216 24.5 / 40.0; columns at multiples of 32 bytes 25.5 / 16.6, 109 / 86) |
                              // kPermOnce (a block's lines of the tensor are all its own, or nearly: the gather's loads
                              // of them may stream; along b: its pieces of the tensor are four lines and more) |
                              // kPermGroups (flat and dense along a: 16 bytes of neighbours along a at a time) |
                              // kPermImageOnce (the same of the image: the scatter's loads of it may stream)
  uint32_t n_slower;          // how many of the other dimensions are slower than a in the image
};
static_assert(sizeof(DsPerm) == 176, "eleven 16-byte words");

struct DsPermItem {
  uint32_t perm, tile;  // which view, which block of it
};

// One block, as the phases need it.  A "row" is the block's part of one step along a; with kPermFlat the
// rows follow each other without a gap in the image and the whole block counts as one row.  Positions are
// 32-bit: tensor offsets count from src0, image offsets from the 16-byte unit that holds the block's first byte.
struct DsPermBlock {
  uint64_t src0;       // tensor address of the block's first element
  uint64_t unit0;      // image offset of the unit that holds the block's first byte
  uint32_t skew;       // where in that unit the byte lies
  uint32_t lo, hi;     // image offsets to move (the call's range, cut to the view's whole units): multiples of 16
  uint32_t da, sa, sb; // distances as in DsPerm
  uint32_t na, nb;     // elements of the block
  uint32_t nbx;        // gather: columns read, up to 15 bytes (wide blocks: 127) more than nb where the next block starts
                       // inside a unit (a line)
  bool first_b, last_b;  // does the block hold the first / the last column of its rows?
  bool inside;         // do all its bytes lie in [lo, hi)?
};

DS_PERM_FN uint32_t ds_perm_min(uint32_t a, uint32_t b) { return a < b ? a : b; }

// i / d for i, d < 2^15 with m = 2^32 / d rounded up (d > 1)
DS_PERM_FN uint32_t ds_perm_magic(uint32_t d) { return 0xFFFFFFFFu / d + 1u; }
DS_PERM_FN uint32_t ds_perm_div(uint32_t i, uint32_t d, uint32_t m) {
  return d == 1 ? i : (uint32_t)(((uint64_t)i * m) >> 32);
}

DS_PERM_FN uint32_t ds_perm_offset(uint64_t x, uint64_t from) {  // x - from, cut to 0 .. 2^31
  return x <= from ? 0u : x - from < (1ull << 31) ? (uint32_t)(x - from) : 1u << 31;
}

// Block t of the view; false if none of it lies in image bytes [img_lo, img_hi).
DS_PERM_FN bool ds_perm_block(const DS_PERM_TABLE DsPerm &d, uint32_t t, uint64_t img_lo, uint64_t img_hi, bool pack, DsPermBlock &k) {
  const uint32_t rest = t / d.tiles_b, tb = t - rest * d.tiles_b;
  uint32_t batch = rest / d.tiles_a;
  const uint32_t ta = rest - batch * d.tiles_a;
  uint64_t src0 = d.src, img0 = d.img;
  for (int j = (int)d.n_batch - 1; j >= 0; --j) {
    const uint32_t q = batch / d.bext[j], r = batch - q * d.bext[j];
    src0 += r * d.bsrc[j];
    img0 += r * d.bimg[j];
    batch = q;
  }
  const uint32_t a0 = ta * d.ta, b0 = tb * d.tb;
  k.src0 = src0 + a0 * d.sa + b0 * d.sb;
  img0 += a0 * d.da + (uint64_t)b0 * d.run;
  k.skew = (uint32_t)img0 & 15u;
  k.unit0 = img0 - k.skew;
  k.da = (uint32_t)d.da;
  k.sa = (uint32_t)d.sa;
  k.sb = (uint32_t)d.sb;
  k.na = ds_perm_min(d.ta, d.ea - a0);
  k.nb = ds_perm_min(d.tb, d.eb - b0);
  k.first_b = b0 == 0;
  k.last_b = b0 + k.nb == d.eb;
  const bool units = ((k.skew | k.da | k.nb * d.run) & 15u) == 0;  // every row is whole 16-byte units
  k.nbx = pack && !k.last_b && !units ? ds_perm_min(k.nb + (14 + d.run) / d.run, d.eb - b0) : k.nb;
  if (pack && (d.flags & (kPermWide | kPermLines)) == kPermWide)
    k.nbx = ds_perm_min(k.nb + (kPermLine - 1) / d.run, d.eb - b0);
  k.lo = ds_perm_offset(img_lo > d.img ? img_lo : d.img, k.unit0);
  k.hi = ds_perm_offset(img_hi < d.end16 ? img_hi : d.end16, k.unit0);
  const uint32_t end = k.skew + (k.na - 1) * k.da + k.nbx * d.run;
  k.inside = k.skew >= k.lo && end <= k.hi;
  return k.skew < k.hi && end > k.lo;
}

// Where row a of the block starts in the image, and in LDS: a row lies in LDS at the same position inside a
// 16-byte unit as in the image.
DS_PERM_FN uint32_t ds_perm_row_image(const DsPermBlock &k, uint32_t a) { return k.skew + a * k.da; }
DS_PERM_FN uint32_t ds_perm_row_start(const DS_PERM_TABLE DsPerm &d, uint32_t a) {
  return a * d.pitch + (d.flags & kPermWide ? a / 4 * 16 : 0u);
}
DS_PERM_FN uint32_t ds_perm_row_lds(const DS_PERM_TABLE DsPerm &d, const DsPermBlock &k, uint32_t a) {
  if (d.flags & kPermFlat) return ds_perm_row_image(k, a);
  return ds_perm_row_start(d, a) + (ds_perm_row_image(k, a) & 15u);
}

// ---- tensor side: granules of type E -------------------------------------------------------------------
// Addresses are the block's (one for the work-group) plus a 32-bit offset.  Gather: every load of a batch is
// issued before the first is used; indices beyond the block are pulled back to its last element, which is then
// moved twice, so that no load hangs on a condition.  Scatter: only what lies in [lo, hi) is stored.
template <typename T, bool NT = false>
DS_PERM_FN T ds_perm_load(uint64_t base, uint32_t off, uint32_t align) {
  DS_PERM_TOUCH(NT ? 's' : 'r', base + off, sizeof(T), align);
  T v;
#if defined(__HIP_DEVICE_COMPILE__)
  typedef T any __attribute__((aligned(1)));
  if (NT) v = __builtin_nontemporal_load((const DS_PERM_GLOBAL any *)(base + off));
  else v = *(const DS_PERM_GLOBAL any *)(base + off);
#else
  memcpy(&v, (const void *)(uintptr_t)(base + off), sizeof(T));
#endif
  (void)align;
  return v;
}
template <typename T, bool NT = false>
DS_PERM_FN void ds_perm_store(uint64_t base, uint32_t off, T v, uint32_t align) {
  DS_PERM_TOUCH('w', base + off, sizeof(T), align);
#if defined(__HIP_DEVICE_COMPILE__)
  typedef T any __attribute__((aligned(1)));
  if (NT) __builtin_nontemporal_store(v, (DS_PERM_GLOBAL any *)(base + off));
  else *(DS_PERM_GLOBAL any *)(base + off) = v;
#else
  memcpy((void *)(uintptr_t)(base + off), &v, sizeof(T));
#endif
  (void)align;
}
// 12 bytes at a multiple of 4
struct DsPermRun {
  uint32_t w[3];
};
#if defined(__HIP_DEVICE_COMPILE__)
typedef uint32_t DsPermThree __attribute__((ext_vector_type(3)));
typedef DsPermThree DsPermThreeAny __attribute__((aligned(4)));
#endif
template <bool NT>
DS_PERM_FN DsPermRun ds_perm_load_run(uint64_t base, uint32_t off) {
  DS_PERM_TOUCH(NT ? 's' : 'r', base + off, 12, 4);
  DsPermRun v;
#if defined(__HIP_DEVICE_COMPILE__)
  DsPermThree x;
  if (NT) x = __builtin_nontemporal_load((const DS_PERM_GLOBAL DsPermThreeAny *)(base + off));
  else x = *(const DS_PERM_GLOBAL DsPermThreeAny *)(base + off);
  v = DsPermRun{{x.x, x.y, x.z}};
#else
  memcpy(v.w, (const void *)(uintptr_t)(base + off), 12);
#endif
  return v;
}
DS_PERM_FN void ds_perm_store_run(uint64_t base, uint32_t off, const DsPermRun &v) {
  DS_PERM_TOUCH('w', base + off, 12, 4);
#if defined(__HIP_DEVICE_COMPILE__)
  *(DS_PERM_GLOBAL DsPermThreeAny *)(base + off) = DsPermThree{v.w[0], v.w[1], v.w[2]};
#else
  memcpy((void *)(uintptr_t)(base + off), v.w, 12);
#endif
}
// Around streaming accesses: an opaque offset in front, a mark behind loads.  (Of two loops that differ in the cache policy
// alone the compiler makes one, with cached accesses.)
template <bool NT>
DS_PERM_FN uint32_t ds_perm_apart(uint32_t off) {
#if defined(__HIP_DEVICE_COMPILE__)
  if (NT) asm volatile("" : "+v"(off));
#endif
  return off;
}
template <bool NT>
DS_PERM_FN void ds_perm_loaded() {
#if defined(__HIP_DEVICE_COMPILE__)
  if (NT) asm volatile("; streamed");
#endif
}
template <typename E>
DS_PERM_FN E ds_perm_get(const uint8_t *lds, uint32_t at) {
  DS_PERM_TOUCH('l', at, sizeof(E), sizeof(E));
  return *(const E *)(lds + at);
}
template <typename E>
DS_PERM_FN void ds_perm_put(uint8_t *lds, uint32_t at, E v) {
  DS_PERM_TOUCH('l', at, sizeof(E), sizeof(E));
  *(E *)(lds + at) = v;
}

typedef uint32_t DsPermQuad __attribute__((vector_size(16)));
// Element e of 16 bytes
template <typename E>
DS_PERM_FN E ds_perm_element(const DsPermQuad &v, uint32_t e) {
  if (sizeof(E) == 8) return (E)(v[2 * e & 3] | (uint64_t)v[(2 * e + 1) & 3] << 32);
  return (E)(v[e * sizeof(E) / 4] >> (8 * (e * sizeof(E) & 3)));
}
template <typename E>
DS_PERM_FN void ds_perm_set_element(uint32_t *w, uint32_t e, E x) {
  if (sizeof(E) == 8) {
    w[2 * e & 3] = (uint32_t)x;
    w[(2 * e + 1) & 3] = (uint32_t)((uint64_t)x >> 32);
  } else {
    w[e * sizeof(E) / 4] |= (uint32_t)x << (8 * (e * sizeof(E) & 3));
  }
}

// Walk along a, the usual block: ds_perm_full_a<E>() steps along a, one granule per run.  Neighbouring threads take
// neighbours along a, V granules of type E each as one access of type W (V > 1: dense along a, whole groups of V);
// a thread goes down b at a fixed step, so that its places in LDS are its first one plus constants.  LDS rows have
// room for whole batches: columns beyond the block are loaded from its last one and never used (the plan takes this
// walk only where a whole batch of columns lies at 32-bit offsets).
template <typename E, typename W, bool PACK>
DS_PERM_FN void ds_perm_full(const DS_PERM_TABLE DsPerm &d, const DsPermBlock &k, uint8_t *lds, uint32_t tid) {
  constexpr uint32_t S = (uint32_t)sizeof(E), V = (uint32_t)(sizeof(W) / sizeof(E));
  constexpr uint32_t lanes = ds_perm_full_a(S) / V, step = kPermThreads / lanes;
  constexpr int U = ds_perm_full_b(S) / step < 16 ? ds_perm_full_b(S) / step : 16;
  const uint32_t n_cols = PACK ? k.nbx : k.nb;
  const uint32_t a = (tid & (lanes - 1)) * V, ac = ds_perm_min(a, k.na - V);
  const uint32_t first = ac * k.sa, last = first + (n_cols - 1) * k.sb;
  uint32_t row[V];
#pragma unroll
  for (uint32_t i = 0; i < V; ++i) row[i] = ds_perm_row_lds(d, k, ac + i) + (tid / lanes) * S;
  if (PACK) {
#pragma unroll 1
    for (uint32_t b0 = 0; b0 < n_cols; b0 += U * step) {
      W v[U];
      uint32_t off = first + (b0 + tid / lanes) * k.sb;
#pragma unroll
      for (int j = 0; j < U; ++j, off += step * k.sb) v[j] = ds_perm_load<W>(k.src0, ds_perm_min(off, last), S);
#pragma unroll
      for (int j = 0; j < U; ++j)
#pragma unroll
        for (uint32_t i = 0; i < V; ++i)
          ds_perm_put<E>(lds, row[i] + b0 * S + (uint32_t)j * step * S, (E)(v[j] >> (8 * S * i)));
    }
  } else if (a < k.na) {
    // the columns whose bytes lie in [lo, hi): granules are never cut
    const uint32_t image = ds_perm_row_image(k, ac);
    const uint32_t c0 = k.inside || k.lo <= image ? 0u : (k.lo - image + S - 1) / S;
    const uint32_t c1 = k.inside ? n_cols : k.hi <= image ? 0u : ds_perm_min((k.hi - image) / S, n_cols);
#pragma unroll 4
    for (uint32_t c = tid / lanes; c < c1; c += step) {
      W v = 0;
#pragma unroll
      for (uint32_t i = 0; i < V; ++i) v |= (W)((W)ds_perm_get<E>(lds, row[i] + (c - tid / lanes) * S) << (8 * S * i));
      if (c >= c0) ds_perm_store<W>(k.src0, first + c * k.sb, v, S);
    }
  }
}

// Walk along a, any block (d.ta is a power of two).
template <typename E, bool PACK, bool NT>
DS_PERM_FN void ds_perm_along_a(const DS_PERM_TABLE DsPerm &d, const DsPermBlock &k, uint8_t *lds, uint32_t tid) {
  const uint32_t n_cols = PACK ? k.nbx : k.nb;
  const uint32_t step = kPermThreads / d.ta, a = tid & (d.ta - 1), ac = ds_perm_min(a, k.na - 1);
  const uint32_t first = ds_perm_apart<NT>(ac * k.sa), row = ds_perm_row_lds(d, k, ac);
  const uint32_t image = ds_perm_row_image(k, ac);
#pragma unroll 1
  for (uint32_t b = tid / d.ta; b < n_cols; b += kPermUnroll * step)
#pragma unroll 1
    for (uint32_t in_run = 0; in_run < d.run; in_run += (uint32_t)sizeof(E)) {
      if (PACK) {
        E v[kPermUnroll];
#pragma unroll
        for (int j = 0; j < kPermUnroll; ++j) {
          const uint32_t c = ds_perm_min(b + (uint32_t)j * step, n_cols - 1);
          v[j] = ds_perm_load<E, NT>(k.src0, first + c * k.sb + in_run, sizeof(E));
        }
        ds_perm_loaded<NT>();
#pragma unroll
        for (int j = 0; j < kPermUnroll; ++j) {
          const uint32_t c = ds_perm_min(b + (uint32_t)j * step, n_cols - 1);
          ds_perm_put<E>(lds, row + c * d.run + in_run, v[j]);
        }
      } else {
#pragma unroll
        for (int j = 0; j < kPermUnroll; ++j) {
          const uint32_t c = b + (uint32_t)j * step, in_row = c * d.run + in_run;
          if (a < k.na && c < n_cols && (k.inside || (image + in_row >= k.lo && image + in_row < k.hi)))
            ds_perm_store<E>(k.src0, first + c * k.sb + in_run, ds_perm_get<E>(lds, row + in_row), sizeof(E));
        }
      }
    }
}

// Walk along b: granule i of the block, rows one behind the other.
template <typename E, bool PACK, bool NT>
DS_PERM_FN void ds_perm_along_b(const DS_PERM_TABLE DsPerm &d, const DsPermBlock &k, uint8_t *lds, uint32_t tid) {
  const uint32_t K = d.run / (uint32_t)sizeof(E);
  const uint32_t per_row = (PACK ? k.nbx : k.nb) * K, total = k.na * per_row;
  const uint32_t m_row = ds_perm_magic(per_row > 1 ? per_row : 2), m_run = ds_perm_magic(K > 1 ? K : 2);
#pragma unroll 1
  for (uint32_t i = tid; i < total; i += kPermUnroll * kPermThreads) {
    uint32_t from[kPermUnroll], at[kPermUnroll], image[kPermUnroll];
#pragma unroll
    for (int j = 0; j < kPermUnroll; ++j) {
      const uint32_t x = ds_perm_min(i + (uint32_t)j * kPermThreads, total - 1);
      const uint32_t a = ds_perm_div(x, per_row, m_row), r = x - a * per_row;
      const uint32_t c = ds_perm_div(r, K, m_run);
      const uint32_t in_row = r * (uint32_t)sizeof(E);  // the granules of a row are dense in the image
      from[j] = a * k.sa + c * k.sb + (r - c * K) * (uint32_t)sizeof(E);
      at[j] = ds_perm_row_lds(d, k, a) + in_row;
      image[j] = ds_perm_row_image(k, a) + in_row;
    }
    if (PACK) {
      E v[kPermUnroll];
#pragma unroll
      for (int j = 0; j < kPermUnroll; ++j) v[j] = ds_perm_load<E, NT>(k.src0, ds_perm_apart<NT>(from[j]), sizeof(E));
#pragma unroll
      for (int j = 0; j < kPermUnroll; ++j) ds_perm_put<E>(lds, at[j], v[j]);
    } else {
#pragma unroll
      for (int j = 0; j < kPermUnroll; ++j)
        if (i + (uint32_t)j * kPermThreads < total && (k.inside || (image[j] >= k.lo && image[j] < k.hi)))
          ds_perm_store<E>(k.src0, from[j], ds_perm_get<E>(lds, at[j]), sizeof(E));
    }
  }
}

// Walk along b, runs of 12 bytes: a run is one access, and its place takes one division and not two for each granule.
// (150 MB of six of every sixteen bf16, us: granule by granule 103 / 192, now 97 / 190, in smaller blocks 87 / 181; 12 MB 12.0 /
// 13.2, now 9.7 / 11.8.  As three accesses of 4 bytes, each on as many lines, 138; so runs of 3 granules of 2 bytes stay
// granule by granule.)
template <bool PACK, bool NT>
DS_PERM_FN void ds_perm_runs(const DS_PERM_TABLE DsPerm &d, const DsPermBlock &k, uint8_t *lds, uint32_t tid) {
  typedef uint32_t E;
  constexpr int U = PACK ? 6 : 4;
  const uint32_t per_row = PACK ? k.nbx : k.nb, total = k.na * per_row, m_row = ds_perm_magic(per_row > 1 ? per_row : 2);
#pragma unroll 1
  for (uint32_t i = tid; i < total; i += U * kPermThreads) {
    uint32_t from[U], at[U], image[U];
    DsPermRun v[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const uint32_t x = ds_perm_min(i + (uint32_t)j * kPermThreads, total - 1);
      const uint32_t a = ds_perm_div(x, per_row, m_row), c = x - a * per_row;
      from[j] = a * k.sa + c * k.sb;
      at[j] = ds_perm_row_lds(d, k, a) + c * 12;
      image[j] = ds_perm_row_image(k, a) + c * 12;
    }
    if (PACK) {
#pragma unroll
      for (int j = 0; j < U; ++j) v[j] = ds_perm_load_run<NT>(k.src0, ds_perm_apart<NT>(from[j]));
#pragma unroll
      for (int j = 0; j < U; ++j)
#pragma unroll
        for (uint32_t g = 0; g < 3; ++g) ds_perm_put<E>(lds, at[j] + 4 * g, v[j].w[g]);
    } else {
#pragma unroll
      for (int j = 0; j < U; ++j)
#pragma unroll
        for (uint32_t g = 0; g < 3; ++g) v[j].w[g] = ds_perm_get<E>(lds, at[j] + 4 * g);
#pragma unroll
      for (int j = 0; j < U; ++j) {
        if (i + (uint32_t)j * kPermThreads >= total) break;
        if (k.inside) {
          ds_perm_store_run(k.src0, from[j], v[j]);
        } else {
#pragma unroll
          for (uint32_t g = 0; g < 3; ++g)
            if (image[j] + 4 * g >= k.lo && image[j] + 4 * g < k.hi) ds_perm_store<E>(k.src0, from[j] + 4 * g, v[j].w[g], 4);
        }
      }
    }
  }
}

// The first n < 16 bytes of w to p, as at most four pieces.  (The ends of rows that are not whole units.)
template <char KIND, typename T>
DS_PERM_FN void ds_perm_put_piece(uint64_t p, T v, uint32_t align) {
  DS_PERM_TOUCH(KIND, p, sizeof(T), align);
#if defined(__HIP_DEVICE_COMPILE__)
  typedef T any __attribute__((aligned(1)));
  *(DS_PERM_GLOBAL any *)p = v;
#else
  memcpy((void *)(uintptr_t)p, &v, sizeof(T));
#endif
  (void)align;
}
template <uint32_t S, char KIND = 'i'>
DS_PERM_FN void ds_perm_put_bytes(uint64_t p, uint32_t n, const uint32_t *w) {
  uint64_t v = w[0] | (uint64_t)w[1] << 32;
  if (n & 8) {
    ds_perm_put_piece<KIND, uint64_t>(p, v, S);
    p += 8;
    v = w[2] | (uint64_t)w[3] << 32;
  }
  if (S <= 4 && (n & 4)) {
    ds_perm_put_piece<KIND, uint32_t>(p, (uint32_t)v, S);
    p += 4;
    v >>= 32;
  }
  if (S <= 2 && (n & 2)) {
    ds_perm_put_piece<KIND, uint16_t>(p, (uint16_t)v, S);
    p += 2;
    v >>= 16;
  }
  if (S <= 1 && (n & 1)) ds_perm_put_piece<KIND, uint8_t>(p, (uint8_t)v, 1);
}

// ---- flat blocks dense along a (kPermGroups), tensor side ----
// 16 bytes of neighbours along a at a time, group by group along a and column by column.  Gather: where the block is no
// whole number of groups, each column's last one is pulled back and moves some elements twice; the scatter stores the
// elements behind the last whole group, and in front of the view's cut unit, in at most four pieces.  Blocks of equal length, as
// few as fit: in powers of two, one element per thread and column, 536 x 536 x 9 fp32 channels-last (155 MB of them, us) 76.7 / 88.5, now 54.5 / 63.8 (a plain copy
// 48.5), one of 10 MB 7.6 / 9.5, now 6.2 / 7.1; transposed bytes 256 x 265 (54 MB) 28.2 / 40.2, now 20.6 / 30.9.
template <typename E, bool PACK, bool NT>
DS_PERM_FN void ds_perm_groups(const DS_PERM_TABLE DsPerm &d, const DsPermBlock &k, uint8_t *lds, uint32_t tid) {
  constexpr uint32_t S = (uint32_t)sizeof(E), G = 16 / S;
  constexpr int U = PACK ? 4 : 2;
  const uint32_t groups = (k.na + G - 1) / G, total = groups * k.nb, m = ds_perm_magic(groups > 1 ? groups : 2);
#pragma unroll 1
  for (uint32_t i = tid; i < total; i += U * kPermThreads) {
    uint32_t from[U], at[U], a[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const uint32_t x = ds_perm_min(i + (uint32_t)j * kPermThreads, total - 1);
      const uint32_t c = ds_perm_div(x, groups, m);
      a[j] = (x - c * groups) * G;
      if (PACK) a[j] = ds_perm_min(a[j], k.na - G);
      from[j] = a[j] * S + c * k.sb;
      at[j] = k.skew + a[j] * k.da + c * S;
    }
    if (PACK) {
      DsPermQuad v[U];
#pragma unroll
      for (int j = 0; j < U; ++j) v[j] = ds_perm_load<DsPermQuad, NT>(k.src0, ds_perm_apart<NT>(from[j]), S);
      ds_perm_loaded<NT>();
#pragma unroll
      for (int j = 0; j < U; ++j)
#pragma unroll
        for (uint32_t e = 0; e < G; ++e) ds_perm_put<E>(lds, at[j] + e * k.da, ds_perm_element<E>(v[j], e));
    } else {
#pragma unroll
      for (int j = 0; j < U; ++j) {
        if (i + (uint32_t)j * kPermThreads >= total) break;
        uint32_t n = ds_perm_min(k.na - a[j], G);
        if (!k.inside) {  // (a row's elements are da apart in the image, none is cut by the range)
          if (k.hi <= at[j]) continue;
          n = ds_perm_min(n, (k.hi - at[j] + k.da - 1) / k.da);
          if (k.lo > at[j]) {
            for (uint32_t e = (k.lo - at[j] + k.da - 1) / k.da; e < n; ++e)
              ds_perm_store<E>(k.src0, from[j] + e * S, ds_perm_get<E>(lds, at[j] + e * k.da), S);
            continue;
          }
        }
        uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
        for (uint32_t e = 0; e < G; ++e) ds_perm_set_element<E>(w, e, ds_perm_get<E>(lds, at[j] + ds_perm_min(e, n - 1) * k.da));
        if (n == G) ds_perm_store<DsPermQuad>(k.src0, from[j], DsPermQuad{w[0], w[1], w[2], w[3]}, S);
        else ds_perm_put_bytes<S, 'w'>(k.src0 + from[j], n * S, w);
      }
    }
  }
}

// ---- wide blocks, tensor side ----
// A thread takes 8 columns of 16 bytes along a and transposes them in registers: its loads, its stores and its accesses
// of LDS are 16 bytes each (bytes: LDS 8).  In LDS row a starts at ds_perm_row_start: an odd number of 16-byte words
// apart, one more after every fourth, which puts the words that 16 neighbouring lanes write into different banks.
// LDS accesses of type T at ALIGN bytes
template <typename T, uint32_t ALIGN>
DS_PERM_FN T ds_perm_lds_load(const uint8_t *lds, uint32_t at) {
  DS_PERM_TOUCH('l', at, sizeof(T), ALIGN);
#if defined(__HIP_DEVICE_COMPILE__)
  typedef T aligned_so __attribute__((aligned(ALIGN)));
  return *(const aligned_so *)(lds + at);
#else
  T v;
  memcpy(&v, lds + at, sizeof(T));
  return v;
#endif
}
template <typename T>
DS_PERM_FN void ds_perm_lds_store(uint8_t *lds, uint32_t at, T v) {
  DS_PERM_TOUCH('l', at, sizeof(T), sizeof(T));
#if defined(__HIP_DEVICE_COMPILE__)
  *(T *)(lds + at) = v;
#else
  memcpy(lds + at, &v, sizeof(T));
#endif
}

// bytes of hi || lo (lo: bytes 0..3), picked by the four bytes of sel
DS_PERM_FN uint32_t ds_perm_pick(uint32_t hi, uint32_t lo, uint32_t sel) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_perm(hi, lo, sel);
#else
  const uint64_t both = (uint64_t)hi << 32 | lo;
  uint32_t r = 0;
  for (int i = 0; i < 4; ++i) r |= (uint32_t)(both >> (8 * (sel >> (8 * i) & 7u)) & 0xFFu) << (8 * i);
  return r;
#endif
}

// Word w of row x of the transposed of `in`, rows of W words with elements of S bytes.
template <uint32_t S, int W>
DS_PERM_FN uint32_t ds_perm_word(const uint32_t (*in)[W], int x, int w) {
  if (S == 8) return in[w / 2][2 * x + (w & 1)];
  if (S == 4) return in[w][x];
  if (S == 2) return ds_perm_pick(in[2 * w + 1][x / 2], in[2 * w][x / 2], x & 1 ? 0x07060302u : 0x05040100u);
  const int c = x / 4;
  const uint32_t pair = x & 2 ? 0x07030602u : 0x05010400u;  // two bytes of two rows
  const uint32_t p = ds_perm_pick(in[4 * w + 1][c], in[4 * w][c], pair);
  const uint32_t q = ds_perm_pick(in[4 * w + 3][c], in[4 * w + 2][c], pair);
  return ds_perm_pick(q, p, x & 1 ? 0x07060302u : 0x05040100u);
}

// N words from any byte of LDS (S = 4, 8: any word)
template <uint32_t S, int N>
DS_PERM_FN void ds_perm_lds_words(const uint8_t *lds, uint32_t at, uint32_t *out) {
  static_assert(N == 2 || N % 4 == 0, "whole quads, or two words");
  const uint32_t from = at & ~3u;
  uint32_t v[N + 1];
  if (N == 2) {
    v[0] = ds_perm_lds_load<uint32_t, 4>(lds, from);
    v[1] = ds_perm_lds_load<uint32_t, 4>(lds, from + 4);
  } else {
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
      const DsPermQuad q = ds_perm_lds_load<DsPermQuad, 4>(lds, from + 16 * i);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[4 * i + j] = q[j];
    }
  }
  if (S >= 4) {
#pragma unroll
    for (int i = 0; i < N; ++i) out[i] = v[i];
    return;
  }
  v[N] = ds_perm_lds_load<uint32_t, 4>(lds, from + 4 * N);
#pragma unroll
  for (int i = 0; i < N; ++i) out[i] = ds_align_bytes(v[i + 1], v[i], at & 3u);
}

template <uint32_t S, bool NT>
DS_PERM_FN void ds_perm_wide_columns(const uint32_t (*in)[2 * S], const DsPermBlock &k, uint32_t off, uint32_t c) {
  off = ds_perm_apart<NT>(off);
#pragma unroll
  for (int j = 0; j < 8; ++j, off += k.sb)
    if (c + j < k.nb)
      ds_perm_store<DsPermQuad, NT>(k.src0, off, DsPermQuad{ds_perm_word<S>(in, j, 0), ds_perm_word<S>(in, j, 1),
                                                            ds_perm_word<S>(in, j, 2), ds_perm_word<S>(in, j, 3)}, S);
}

template <typename E, bool PACK, bool NT>
DS_PERM_FN void ds_perm_wide(const DS_PERM_TABLE DsPerm &d, const DsPermBlock &k, uint8_t *lds, uint32_t tid) {
  constexpr uint32_t S = (uint32_t)sizeof(E), G = 16 / S, lanes = kPermWideA / G;
  constexpr int W = 2 * S;  // words of 8 elements
  const uint32_t a = tid % lanes * G, c = tid / lanes * 8, n_cols = PACK ? k.nbx : k.nb;
  if (a >= k.na || c >= n_cols) return;
  const uint32_t first = a * S + c * k.sb, last = a * S + (n_cols - 1) * k.sb;
  if (PACK) {
    uint32_t in[8][4], off = ds_perm_apart<NT>(first);
#pragma unroll
    for (int j = 0; j < 8; ++j, off += k.sb) {  // columns beyond the block: its last one again
      const DsPermQuad q = ds_perm_load<DsPermQuad, NT>(k.src0, ds_perm_min(off, last), S);
#pragma unroll
      for (int w = 0; w < 4; ++w) in[j][w] = q[w];
    }
    ds_perm_loaded<NT>();
#pragma unroll
    for (uint32_t i = 0; i < G; ++i) {
      const uint32_t at = ds_perm_row_start(d, a + i) + c * S;
      if (S == 1) {
        ds_perm_lds_store(lds, at, ds_perm_word<S>(in, i, 0) | (uint64_t)ds_perm_word<S>(in, i, 1) << 32);
      } else {
#pragma unroll
        for (int u = 0; u < W; u += 4) {
          if (u && c + u * 4 / S >= n_cols) break;
          ds_perm_lds_store(lds, at + 4 * u, DsPermQuad{ds_perm_word<S>(in, i, u), ds_perm_word<S>(in, i, u + 1),
                                                        ds_perm_word<S>(in, i, u + 2), ds_perm_word<S>(in, i, u + 3)});
        }
      }
    }
  } else {
    uint32_t in[G][W];
#pragma unroll
    for (uint32_t i = 0; i < G; ++i) ds_perm_lds_words<S, W>(lds, ds_perm_row_lds(d, k, a + i) + c * S, in[i]);
    if (d.flags & kPermStream) ds_perm_wide_columns<S, true>(in, k, first, c);
    else ds_perm_wide_columns<S, false>(in, k, first, c);
  }
}

// STREAM: the image is one of those that no cache holds until the next pass (kCachedBytes); the gather's loads then stream
// where no line of the tensor is another block's too (kPermOnce).  Walks along b, streaming / cached, us: pieces of 8 bytes
// that 16 blocks' lines hold (bf16 4096 x 4096 x 4 with strides of 8, 32768 and 2) 301 / 155, of 24 bytes (1500 x 3000 x 6
// with strides of 16, 24 000 and 2) 189 / 108, of 16 bytes of bytes 127 / 90; long pieces, which share the lines at their
// ends alone, 39.6 / 43.6 (fp32, every second of 1000 columns), 45.8 / 48.4 (bf16, of 1031), 44.0 / 48.7 (six of sixteen).
template <typename E, typename W, bool PACK, bool STREAM = false>
DS_PERM_FN void ds_perm_tensor_side(const DS_PERM_TABLE DsPerm &d, const DsPermBlock &k, uint8_t *lds, uint32_t tid) {
  constexpr uint32_t V = (uint32_t)(sizeof(W) / sizeof(E));
  constexpr bool NT = PACK && STREAM;
  const bool once = NT && (d.flags & kPermOnce);
  if constexpr (sizeof(E) == 4)
    if (!(d.flags & kPermAlongA) && d.run == 12) {
      if (once) ds_perm_runs<PACK, NT>(d, k, lds, tid);
      else ds_perm_runs<PACK, false>(d, k, lds, tid);
      return;
    }
  if (d.flags & kPermGroups) {
    if (PACK && k.na < 16 / sizeof(E)) ds_perm_along_b<E, PACK, false>(d, k, lds, tid);
    else if (once) ds_perm_groups<E, PACK, NT>(d, k, lds, tid);
    else ds_perm_groups<E, PACK, false>(d, k, lds, tid);
  } else if ((d.flags & kPermWide) && (PACK || k.inside)) {
    if (once) ds_perm_wide<E, PACK, NT>(d, k, lds, tid);
    else ds_perm_wide<E, PACK, false>(d, k, lds, tid);
  } else if (!(d.flags & kPermAlongA)) {
    if (once) ds_perm_along_b<E, PACK, NT>(d, k, lds, tid);
    else ds_perm_along_b<E, PACK, false>(d, k, lds, tid);
  } else if (!(d.flags & kPermFull)) {
    if (once) ds_perm_along_a<E, PACK, NT>(d, k, lds, tid);
    else ds_perm_along_a<E, PACK, false>(d, k, lds, tid);
  } else if (V > 1 && d.sa == sizeof(E) && k.na % V == 0 && (PACK || k.inside)) {
    ds_perm_full<E, W, PACK>(d, k, lds, tid);
  } else {
    ds_perm_full<E, E, PACK>(d, k, lds, tid);
  }
}

// ---- image side ---------------------------------------------------------------------------------------------
// The bytes of the row a work-group writes (gather), relative to the start of the 16-byte unit that holds the
// row's first byte.  Inside a row, blocks meet at unit boundaries, so a unit is written whole by one block;
// only where a row starts or ends inside a unit are its two parts written by two rows.
DS_PERM_FN void ds_perm_window(const DS_PERM_TABLE DsPerm &d, const DsPermBlock &k, uint32_t unit, uint32_t skew, uint32_t &w0,
                               uint32_t &w1) {
  if (d.flags & kPermFlat) {
    w0 = skew;
    w1 = skew + k.na * k.da;
  } else if (d.flags & kPermWide) {
    // ... at line boundaries of the image
    const uint32_t read_end = skew + k.nbx * d.run, line = (uint32_t)(k.unit0 + unit) & (kPermLine - 1);
    w0 = k.first_b ? skew : ds_perm_min(((line + skew + kPermLine - 1) & ~(kPermLine - 1)) - line, read_end);
    w1 = k.last_b ? read_end
                  : ds_perm_min(((line + skew + k.nb * d.run + kPermLine - 1) & ~(kPermLine - 1)) - line, read_end);
  } else {
    const uint32_t read_end = skew + k.nbx * d.run;
    w0 = k.first_b ? skew : ds_perm_min((skew + 15u) & ~15u, read_end);
    w1 = k.last_b ? read_end : ds_perm_min((skew + k.nb * d.run + 15u) & ~15u, read_end);
  }
  if (k.inside) return;
  if (k.lo > unit + w0) w0 = k.lo - unit < w1 ? k.lo - unit : w1;
  if (k.hi < unit + w1) w1 = k.hi > unit ? k.hi - unit : 0u;
}

struct DsPermUnit {
  uint32_t w[4];
};

// Gather: LDS -> image, `img` pointing at image byte img_lo.
// Wide blocks: 32 threads have room for a row's window, which is at most 31 units; four rows' units are read before the first
// is stored.  The parts of units at the ends of rows go last, one for each of two threads per row.  (Row after row, each with
// its whole units or its parts, a block was a chain of eight such steps, which is what a small view takes: transposed bf16,
// 512 x 519, 5.8 us, now 4.7, 512 x 512 4.6 and 4.4, 1000 x 1007 6.0 and 4.9, 80 of those 67.8 and 65.9, bytes 4096 x 4120 (169
// MB) 68.0 and 65.7.)
template <typename E, typename StoreUnit>
DS_PERM_FN void ds_perm_wide_store(const DS_PERM_TABLE DsPerm &d, const DsPermBlock &k, const uint8_t *lds, uint64_t base, uint32_t tid,
                                   StoreUnit store_unit) {
  constexpr uint32_t S = (uint32_t)sizeof(E), U = 4, kNone = ~0u;
#pragma unroll 1
  for (uint32_t first = tid / 32; first < k.na; first += 8 * U) {
    DsPermUnit v[U];
    uint32_t to[U];
#pragma unroll
    for (uint32_t i = 0; i < U; ++i) {
      const uint32_t a = first + 8 * i;
      const uint32_t at = ds_perm_row_image(k, a), skew = at & 15u, unit = at - skew;
      uint32_t w0, w1;
      ds_perm_window(d, k, unit, skew, w0, w1);
      const uint32_t x = (w0 & ~15u) + 16u * (tid & 31u);
      to[i] = a < k.na && x >= w0 && x + 16u <= w1 ? unit + x : kNone;
      if (to[i] != kNone) ds_perm_lds_words<S, 4>(lds, ds_perm_row_start(d, a) + x - skew, v[i].w);
    }
#pragma unroll
    for (uint32_t i = 0; i < U; ++i)
      if (to[i] != kNone) {
        DS_PERM_TOUCH('i', base + to[i], 16, 16);
        store_unit(base + to[i], v[i]);
      }
  }
  const uint32_t a = tid / 2;
  if (a >= k.na) return;
  const uint32_t at = ds_perm_row_image(k, a), skew = at & 15u, unit = at - skew;
  uint32_t w0, w1;
  ds_perm_window(d, k, unit, skew, w0, w1);
  const uint32_t head = (w0 + 15u) & ~15u;  // where the first whole unit starts
  const uint32_t from = tid & 1u ? (w1 & ~15u) : w0, to = tid & 1u ? w1 : ds_perm_min(head, w1);
  if (from < to && (!(tid & 1u) || from >= head)) {
    DsPermUnit v;
    ds_perm_lds_words<S, 4>(lds, ds_perm_row_start(d, a) + from - skew, v.w);
    ds_perm_put_bytes<S>(base + (unit + from), to - from, v.w);
  }
}

template <typename E, typename StoreUnit>
DS_PERM_FN void ds_perm_image_store(const DS_PERM_TABLE DsPerm &d, const DsPermBlock &k, const uint8_t *lds, uint8_t *img, uint64_t img_lo,
                                    uint32_t tid, StoreUnit store_unit) {
  const uint32_t lanes = 1u << d.lanes_log2, rows = d.flags & kPermFlat ? 1u : k.na;
  const uint64_t base = (uint64_t)(uintptr_t)img + (k.unit0 - img_lo);
  if (d.flags & kPermWide) return ds_perm_wide_store<E>(d, k, lds, base, tid, store_unit);
#pragma unroll 1
  for (uint32_t a = tid >> d.lanes_log2; a < rows; a += kPermThreads >> d.lanes_log2) {
    const uint32_t at = ds_perm_row_image(k, a), skew = at & 15u, unit = at - skew, row = a * d.pitch;
    uint32_t w0, w1;
    ds_perm_window(d, k, unit, skew, w0, w1);
    for (uint32_t x = (w0 & ~15u) + 16u * (tid & (lanes - 1)); x < w1; x += 16u * lanes) {
      if (x >= w0 && x + 16u <= w1) {
        DsPermUnit v;
        DS_PERM_TOUCH('l', row + x, 16, 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) v.w[j] = *(const uint32_t *)(lds + row + x + 4 * j);
        DS_PERM_TOUCH('i', base + (unit + x), 16, 16);
        store_unit(base + (unit + x), v);
      } else {
        const uint32_t x1 = ds_perm_min(w1, x + 16u);
        for (uint32_t y = w0 > x ? w0 : x; y < x1; y += (uint32_t)sizeof(E)) {
          DS_PERM_TOUCH('i', base + (unit + y), sizeof(E), sizeof(E));
          *(DS_PERM_GLOBAL E *)(base + (unit + y)) = ds_perm_get<E>(lds, row + y);
        }
      }
    }
  }
}

// Scatter: image -> LDS, every unit of the range that holds bytes of the block's rows.
template <typename LoadUnit>
DS_PERM_FN void ds_perm_image_load(const DS_PERM_TABLE DsPerm &d, const DsPermBlock &k, uint8_t *lds, const uint8_t *img, uint64_t img_lo,
                                   uint32_t tid, LoadUnit load_unit) {
  const uint32_t lanes = 1u << d.lanes_log2, flat = d.flags & kPermFlat, rows = flat ? 1u : k.na;
  const uint64_t base = (uint64_t)(uintptr_t)img + (k.unit0 - img_lo);
  if ((d.flags & kPermWide) && k.inside) {  // a thread's units of all its rows at once
    DsPermUnit v[kPermWideA / 8];
#pragma unroll
    for (uint32_t i = 0; i < kPermWideA / 8; ++i) {
      const uint32_t a = ds_perm_min(tid / 32 + 8 * i, k.na - 1);
      const uint32_t at = ds_perm_row_image(k, a), skew = at & 15u, x = 16u * (tid & 31u);
      if (x < skew + k.nb * d.run) {
        DS_PERM_TOUCH('j', base + (at - skew + x), 16, 16);
        v[i] = load_unit(base + (at - skew + x));
      }
    }
#pragma unroll
    for (uint32_t i = 0; i < kPermWideA / 8; ++i) {
      const uint32_t a = ds_perm_min(tid / 32 + 8 * i, k.na - 1);
      const uint32_t skew = ds_perm_row_image(k, a) & 15u, x = 16u * (tid & 31u);
      if (x < skew + k.nb * d.run)
        ds_perm_lds_store(lds, ds_perm_row_start(d, a) + x, DsPermQuad{v[i].w[0], v[i].w[1], v[i].w[2], v[i].w[3]});
    }
    return;
  }
#pragma unroll 1
  for (uint32_t a = tid >> d.lanes_log2; a < rows; a += kPermThreads >> d.lanes_log2) {
    const uint32_t at = ds_perm_row_image(k, a), skew = at & 15u, unit = at - skew, row = ds_perm_row_start(d, a);
    const uint32_t end = skew + (flat ? k.na * k.da : k.nb * d.run);
    for (uint32_t x = 16u * (tid & (lanes - 1)); x < end; x += 16u * lanes) {
      if (unit + x < k.lo || unit + x >= k.hi) continue;
      DS_PERM_TOUCH('j', base + (unit + x), 16, 16);
      const DsPermUnit v = load_unit(base + (unit + x));
      DS_PERM_TOUCH('l', row + x, 16, 4);
#pragma unroll
      for (int j = 0; j < 4; ++j) *(uint32_t *)(lds + row + x + 4 * j) = v.w[j];
    }
  }
}

// ---- the plan's side (host) -----------------------------------------------------------------------------------
// Fills `d` for a view of `n_outer` outer dimensions (slowest first, strides in bytes) of runs of `run` bytes at
// image offset `img`; returns the number of blocks, or 0 if the view is not one of this route's: one contiguous
// run, runs of 16 bytes and more (a unit then lies in at most two runs: the row and general paths move it with
// whole 16-byte accesses), less than kPermMinBytes, extents that leave a block nearly empty or exceed 31 bits.
static inline uint64_t ds_perm_make(uint64_t src, uint64_t img, uint64_t nbytes, uint64_t run, uint32_t n_outer,
                                    const uint64_t *extent, const uint64_t *stride, uint64_t image_bytes, DsPerm *d) {
  if (n_outer == 0 || run >= 16 || nbytes < kPermMinBytes) return 0;
  uint64_t bits = src | run, columns = src;  // `columns`: where those of a view dense along a can start
  for (uint32_t j = 0; j < n_outer; ++j) {
    if (extent[j] >= (1ull << 31)) return 0;
    bits |= stride[j];
    if (stride[j] != run) columns |= stride[j];
  }
  memset(d, 0, sizeof(*d));
  d->src = src;
  d->img = img;
  d->end16 = img + (nbytes & ~(uint64_t)15);
  d->run = (uint32_t)run;
  uint32_t g_log2 = 0;
  while (g_log2 < 3 && !(bits & (1u << g_log2))) ++g_log2;
  const uint32_t g = 1u << g_log2;
  uint64_t image_stride[8];
  uint64_t at = run;
  for (int j = (int)n_outer - 1; j >= 0; --j) {
    image_stride[j] = at;
    at *= extent[j];
  }
  const uint32_t b = n_outer - 1;
  uint32_t a = n_outer;  // the dimension closest in the tensor, the one before b if that is b itself
  for (uint32_t j = 0; j < b; ++j)
    if (stride[j] < stride[b] && (a == n_outer || stride[j] < stride[a])) a = j;
  const bool along_a = a != n_outer;
  if (!along_a && b > 0) a = b - 1;
  d->eb = (uint32_t)extent[b];
  d->sb = stride[b];
  d->ea = a == n_outer ? 1u : (uint32_t)extent[a];
  d->sa = a == n_outer ? 0u : stride[a];
  d->da = a == n_outer ? run * extent[b] : image_stride[a];
  uint64_t batches = 1, image_bits = img | d->da;  // where in a unit rows can start
  for (uint32_t j = 0; j < b; ++j)
    if (j != a) {
      d->bext[d->n_batch] = (uint32_t)extent[j];
      d->bsrc[d->n_batch] = stride[j];
      d->bimg[d->n_batch] = image_stride[j];
      image_bits |= image_stride[j];
      ++d->n_batch;
      if (j < a) ++d->n_slower;
      batches *= extent[j];
    }
  // Rows of less than 512 bytes that are neighbours in the image are taken as one piece, unless they are whole
  // units at unit boundaries anyway.
  const uint64_t row_bytes = run * d->eb;
  const bool neighbours = a == n_outer || a + 1 == b;
  const bool flat = neighbours && row_bytes < 512 && ((row_bytes | img) & 15);
  const bool few = image_bytes <= kPermFewBytes;
  uint32_t ta, tb;
  if (flat) {
    tb = d->eb;
    ta = (uint32_t)(16384 / row_bytes);
    if (!along_a && ta > d->ea) ta = d->ea;
  } else if (along_a) {
    // a line or more along a; along b what 16 KiB leave, less the 15 bytes that rows which are not whole units are
    // read further
    ta = ds_perm_full_a(g);
    while (ta > 1 && ta / 2 >= d->ea) ta /= 2;
    tb = (uint32_t)((16384 / ta) / run);
    if (tb == 0) tb = 1;
    if (tb > d->eb) tb = d->eb;
    else if ((image_bits & 15) && tb * run >= 128) tb -= (uint32_t)((15 + run) / run);
  } else {
    // 8 KiB; bytes, which are 32 granules per thread then, 4 KiB in small images.  us, 16 / 8 / 4 KiB, gather: every second
    // byte, 100 KB 11.7 / 7.3 / 4.9, 2 MB 12.0 / 7.9 / 6.2, 8 MB 16.1 / 12.4 / 13.4, 64 MB 70 / 72 / 84; every third, 100 MB
    // 112 / 110 / 132, scatter 157 / 150 / 143; 16 / 8 KiB: every second fp32, 500 KB 5.3 / 3.9, scatter 5.8 / 4.2, 64 MB in
    // rows of 1000 41.1 / 39.6, scatter 82 / 79.  Rows of 1 KiB and more may be an eighth larger in all, so that a little
    // less room than they take leaves no block nearly empty (every second fp32, 1031 columns, 16 MB: rows cut at 1024 17.5,
    // whole 13.3; 100 MB 99 / 66).  Cut at lines of the image, so that a line is one block's (150 MB of six of
    // sixteen: bytes 108 / 90, at units 107; bf16 97 / 87, at units 93).
    const uint32_t room = g == 1 && few ? 4096 : 8192;
    tb = row_bytes <= 4096 + 512 ? d->eb : (uint32_t)(4096 / run);
    ta = (tb * run >= 1024 ? room + room / 8 : room) / (tb * (uint32_t)run);
    if (ta > d->ea) ta = d->ea;
    if (tb < d->eb) tb = (uint32_t)(room / (ta * run));
    if (tb > d->eb) tb = d->eb;
    if (tb < d->eb) {
      uint32_t whole = 1;  // steps that are whole lines, or whole units
      while ((whole * run) & (image_bits & (kPermLine - 1) ? 15 : kPermLine - 1)) whole *= 2;
      if (tb > whole) tb = tb / whole * whole;
    }
  }
  // flat, dense along a: as few blocks as 16 KiB allow, in small images 8, of equal length, in whole groups of 16 bytes (us, 16
  // / 8 KiB: fp32 with six columns, 1 MB, 3.4 / 3.1, scatter 3.8 / 3.1, 8 MB 4.5 / 4.8 and 5.8 / 5.9; bytes with 60, 350 KB
  // 5.0 / 3.6 and 5.6 / 3.5; fp32 512 x 512 x 9, 9.4 MB, 5.3 / 6.3 and 7.1 / 7.3)
  // Neighbouring threads write LDS 16 bytes' worth of rows apart, which is 4 words for each of the columns: columns in multiples of
  // 4 leave 4 banks or fewer.  That costs nothing where a block has few groups along a, three for each bank (four of
  // 16-bit elements), and is still the better way for rows of 8 bytes or less on 4 banks.  One element per thread and column /
  // groups, gather of 130 MB, us: bytes in 24 columns 77 / 220, 72 columns 72 / 110, 60 columns 67 / 75, 84 columns 0.79 of the time,
  // 200 columns 69 / 52, 4 columns 0.51; bf16 in 20 columns 55 / 62, 28 columns 53 / 60, 100 columns 56 / 47, 4 columns 128 / 66; 12 MB
  // of bf16 in 12 columns 8.4 / 9.6, bytes in 136 columns 1.22 of the time, bf16 in 68 the same.
  bool groups = flat && along_a && run == g && d->sa == g && d->ea >= 16 / g;
  if (groups) {
    const uint32_t G = 16 / g, fit = few ? (uint32_t)(8192 / row_bytes) : ta, most = (fit < ta ? fit : ta) / G * G;
    const uint32_t n = (d->ea + most - 1) / most, even = ((d->ea + n - 1) / n + G - 1) / G;  // blocks, groups of each
    uint32_t banks = 16;
    for (uint32_t c = d->eb; banks > 1 && !(c & 1); c /= 2) banks /= 2;
    if (banks <= 4 && (even < 64 ? even : 64) > (g == 1 ? 3 : 4) * banks && !(banks == 4 && row_bytes <= 8)) groups = false;
    else ta = even * G;
  }
  if (!groups && along_a) {  // a power of two, of at most one step along a per thread
    uint32_t p = 1;
    while (2 * p <= ta && 2 * p <= kPermThreads && p < d->ea) p *= 2;
    ta = p;
  }
  // LDS rows are an odd number of words (of granules of 8 bytes) apart, so that a wavefront's granules along a
  // fall into different banks; a row needs its position inside the unit (up to 15 bytes), the columns up to the
  // next unit (up to 15 bytes and a run more), and whole 16-byte units to its end.
  const uint32_t word = g == 8 ? 8 : 4;
  bool full = along_a && !flat && run == g && ta == ds_perm_full_a(g);
  // ds_perm_full steps through whole batches of columns and pulls what lies beyond the block back to its last one:
  // all of them, in the block or not, must be at 32-bit offsets
  if (full && (d->sa >= (1ull << 31) / ta || d->sb >= (1ull << 31) / ds_perm_full_b(g))) full = false;
  for (;;) {
    uint32_t cols = tb + (uint32_t)((14 + run) / run);
    if (((image_bits | tb * run) & 15) == 0 || tb == d->eb) cols = tb;
    if (full && cols > ds_perm_full_b(g)) full = false;
    if (full) cols = ds_perm_full_b(g);
    d->pitch = (uint32_t)(cols * run + 30 + word - 1) / word * word;
    if (!(d->pitch / word & 1)) d->pitch += word;
    if (flat || ta * d->pitch <= kPermNarrowBytes) break;
    if (full) full = false;
    else if (ta > 1) ta /= 2;
    else return 0;
  }
  // inside a block, positions on either side are 32-bit
  while (ta > 1 && (ta * d->da >= (1ull << 31) || ta * d->sa >= (1ull << 31))) ta /= 2, full = false;
  while (tb > 1 && (uint64_t)(tb + 16) * d->sb >= (1ull << 31)) tb /= 2, full = false;
  if ((uint64_t)(tb + 16) * d->sb >= (1ull << 31) || d->da >= (1ull << 31)) return 0;
  if (flat && tb != d->eb) return 0;
  // Wide blocks, where they have whole 16 bytes along a, and rows of at least four lines
  const bool lines = (image_bits & (kPermLine - 1)) == 0;
  bool wide = along_a && !flat && run == g && d->sa == g && d->ea >= kPermWideA && d->ea % (16 / g) == 0 && row_bytes >= 512;
  if (wide) {
    const uint32_t most = (lines ? kPermWideLines : kPermWideRow) / g, n = (d->eb + most - 1) / most;
    const uint32_t cols = lines ? most : (d->eb + n - 1) / n;
    wide = (cols + kPermLine) * d->sb < (1ull << 31) && kPermWideA * d->da < (1ull << 31);
    if (wide) {
      ta = kPermWideA;
      tb = cols;
      full = false;
      d->pitch = kPermWidePitch;
    }
  }
  if ((uint64_t)(ta < d->ea ? ta : d->ea) * tb * run < kPermMinBytes) return 0;
  d->ta = ta;
  d->tb = tb;
  d->tiles_a = (d->ea + ta - 1) / ta;
  d->tiles_b = (d->eb + tb - 1) / tb;
  const uint32_t units = (uint32_t)((flat ? kPermThreads * 16 : tb * run) / 16);
  while (d->lanes_log2 < 8 && (2u << d->lanes_log2) <= units) ++d->lanes_log2;  // (not used by wide blocks inside the range)
  // Where the scatter's loads stream: wide blocks whose stores do; blocks that are one piece of the image; rows of whole
  // lines, or of at least three.  Of shorter ones another block reads the lines at both ends again, from HBM.  Streaming
  // / cached, scatter, us: rows of 112 bytes (bytes 2273 x 3283, 20 of them) 128 / 94, (5530 x 3933, five) 72 / 64, of 240
  // bytes (bf16 332 941 x 214) 127 / 111, (fp32 37 x 96 x 2230 of 37 x 3552, five) 136 / 118, of 48 bytes (fp32 1000 x 1000
  // x 4 x 3) 90 / 80, though of 240 bytes (fp32 1883 x 2672, five) 49 / 57 too; of 512 (i64 50 x 362, 500 of them) 0.74 of
  // the time, (157 x 97 936) 0.86, of 496 (19 x 307) 0.92; pieces (fp32 660 343 x 6, five) 0.83, (25 x 372 x 372, five) 0.90.
  // Narrow blocks along a store parts of lines of the tensor; beside them the loads stream only as long as the image and the
  // tensors (as many bytes of them for each of the image as this view takes) fit the last-level cache, or seven eighths of it
  // where rows do not start at lines.  Streaming / cached, us: together 144 MB (i64 50 x 362, 500 of them, columns of 50) 31.6 /
  // 36.4, 202 MB (columns of 90) 35.2 / 48.1, 205 MB (24 x 65 537 of 25, eight) 54.8 / 64.0, 249 MB (33 x 515 of 34, 900) 80.3 / 73.6,
  // 302 MB (157 x 20 001 of 158, six) 101.2 / 94.6, 331 MB (fp32 9 x 18 066 of 10, 241) 109 / 101; rows of lines, 246 MB (i64 157 x
  // 97 936) 66.4 / 80.7, 258 MB (fp32 62 x 65 536 of 102, six) 66.5 / 74.4, 292 MB (i64 33 x 100 000 of 40, five) 98.7 / 92.3, 390 MB
  // (33 x 512 of 73, 900) 96.1 / 91.7; but 277 MB (157 x 97 936 of 197) 74.5 / 83.6.
  const bool rows_of_lines = flat || ((image_bits | tb * run) & (kPermLine - 1)) == 0;
  bool image_once = wide ? (columns & 63) == 0 : rows_of_lines || tb * run >= 3 * kPermLine;
  if (along_a && !wide && !flat) {
    uint64_t whole = run;  // bytes from the view's first to its last, or of its batches if these lie apart
    for (uint32_t j = 0; j < n_outer; ++j)
      if (extent[j] * stride[j] > whole) whole = extent[j] * stride[j];
    const uint64_t parts = d->ea * d->sa > d->eb * d->sb ? d->ea * d->sa : d->eb * d->sb;
    const double apart = (double)batches * (double)parts, span = apart < (double)whole ? apart : (double)whole;
    const uint64_t room = rows_of_lines ? kPermCacheBytes : kPermCacheBytes / 8 * 7;
    if ((double)image_bytes * (1.0 + span / (double)nbytes) > (double)room) image_once = false;
  }
  d->flags = g_log2 | (along_a ? kPermAlongA : 0u) | (flat ? kPermFlat : 0u) | (full ? kPermFull : 0u) |
             (groups ? kPermGroups : 0u) | (rows_of_lines ? kPermLines : 0u) | (wide ? kPermWide : 0u) |
             (wide && (columns & 63) == 0 ? kPermStream : 0u) |
             ((wide ? lines && g > 1 && (columns & (kPermLine - 1)) == 0 : (along_a ? ta * d->sa : tb * d->sb) >= 4 * kPermLine) ? kPermOnce : 0u) |
             (image_once ? kPermImageOnce : 0u);
  const unsigned __int128 tiles = (unsigned __int128)batches * d->tiles_a * d->tiles_b;
  return tiles < (1u << 31) ? (uint64_t)tiles : 0;
}

// A launch takes the blocks in image order: by the dimensions slower than a, along a, by the dimensions between a and b,
// along b (ds_perm_block counts along a behind all other dimensions).  Writes the items of a view of n blocks.
static inline void ds_perm_items(const DsPerm &d, uint32_t perm, uint32_t n, DsPermItem *out) {
  uint32_t between = 1;
  for (uint32_t j = d.n_slower; j < d.n_batch; ++j) between *= d.bext[j];
  const uint32_t n_slower = n / (between * d.tiles_a * d.tiles_b);
  for (uint32_t slower = 0; slower < n_slower; ++slower)
    for (uint32_t ta = 0; ta < d.tiles_a; ++ta)
      for (uint32_t x = 0; x < between; ++x)
        for (uint32_t tb = 0; tb < d.tiles_b; ++tb)
          *out++ = {perm, ((slower * between + x) * d.tiles_a + ta) * d.tiles_b + tb};
}

// How a launch's blocks are dealt to the work-groups, of which number w runs on XCD w mod 8: in stripes of neighbouring
// blocks, stripe by stripe over the XCDs, as many for each.  What runs at a time then lies in one part of the tensors and
// of the image, which the DRAM takes better than eight parts far apart, while the lines that neighbouring blocks share
// stay in one L2.  Measured, us, gather / scatter: bf16 4096 x 4120, five of them, one stripe per XCD 64.7 / 64.7, stripes
// of 256 blocks 65.5 / 65.3, 128 63.2 / 62.8, 64 62.4 / 61.5, 32 62.1 / 60.9, single blocks 64.1 / 62.6; bytes of that shape
// 72.8 / 83.2, with stripes of 64 68.3 / 73.6, with single blocks 93.0 / 72.9; the views of perf/cases.py 76.7 / 96.9, with
// stripes 67.5 / 81.6 (kinds of views that take unequal time are dealt evenly too).
// Launches of fewer blocks than about a round of them have one stripe per XCD (gather of 1558 blocks 15.5, in three stripes
// 16.4, of 2035 blocks 19.6 and 20.9; scatter of 625 blocks 9.7, in two 10.9).
struct DsPermOrder {
  uint32_t span;    // work-groups per XCD
  uint32_t stripe;  // blocks of a stripe, at least 2
  uint32_t magic;   // ds_perm_magic of it; 0: one stripe per XCD
};
constexpr uint32_t kPermOrdered = 1u << 27;
// `together`: one stripe per XCD, for launches whose blocks share lines with blocks too far on for a stripe.
// Scatters of mostly narrow blocks along a: their stores of parts of lines wait in the L2 for the others, which are a few
// dozen blocks or the rest of a column further.  In stripes / one per XCD, us: fp32 37 x 96 x 2230 of 37 x 3552, five of them,
// 119 / 99, 1883 x 2672, five, 57 / 54, bf16 332 941 x 214 111 / 105, bytes 2273 x 3283, 20 of them, 94 / 87; but bytes 15 298 x
// 194, five, 0.95 of the time.
// (Wide blocks the other way round: i64 804 x 3735, five, 0.89, bf16 41 282 x 400, five, 0.90.)
// Gathers of mostly walks along b whose lines the next batches read too, kPermFarBlocks blocks and more further: in stripes / one
// per XCD, us, bytes 186 x 37 605 x 9 with strides of 18, 3348 and 2, 21 blocks, 111 / 90, bf16 184 x 59 034 x 2, 15 blocks,
// 140 / 125, 11 x 24 648 x 3, 20 of them, 10 blocks, 66 / 59, fp32 268 x 13 719 x 8, 54 blocks, 109 / 101; nearer ones: two
// blocks, bytes 3000 x 3000 x 8, 90 / 114, bf16 4096 x 4096 x 4 156 / 154, four, fp32 2048 x 2048 x 4, 68 / 64.
constexpr uint32_t kPermFarBlocks = 8;
static inline DsPermOrder ds_perm_order(uint32_t n, bool pack, bool together = false) {  // 0 < n < kPermOrdered
  const uint32_t blocks = 8 * (pack ? 64 : 48);
  const uint32_t rounds = n < (pack ? 2048 : 768) || together ? 1 : (n + blocks / 2) / blocks;
  uint32_t stripe = (n + rounds * 8 - 1) / (rounds * 8);
  if (stripe < 2) stripe = 2;
  return {rounds * stripe, stripe, rounds == 1 ? 0 : ds_perm_magic(stripe)};
}
// The block that work-group w < 8 * span takes; n and more: none.  (Of several stripes per XCD w / 8 * stripe < 2^32: the
// quotient is exact.)
DS_PERM_FN uint32_t ds_perm_ordered(uint32_t w, uint32_t stripe, uint32_t magic) {
  const uint32_t i = w >> 3, round = (uint32_t)(((uint64_t)i * magic) >> 32);
  return (round * 7u + (w & 7u)) * stripe + i;  // stripe 8 round + XCD, block i - round * stripe of it
}

// The blocks [first, last), in that order, that can hold image bytes of [img_lo, img_hi), which holds some of the view's:
// in a launch of a part of the image every block outside it would be a work-group that ends at once, and an image moved
// in n parts would launch n times its blocks (1 GiB of bf16 transposed, 32768 x 16384: gather in 64 parts 7.1 ms, now
// 0.86; whole 0.53).
static inline void ds_perm_range(const DsPerm &d, uint64_t img_lo, uint64_t img_hi, uint64_t *first, uint64_t *last) {
  uint64_t group = d.tiles_b;  // blocks that share their rows along a
  for (uint32_t j = d.n_slower; j < d.n_batch; ++j) group *= d.bext[j];
  const uint64_t lo = img_lo > d.img ? img_lo - d.img : 0, hi = (img_hi < d.end16 ? img_hi : d.end16) - 1 - d.img;
  const uint64_t row_lo = lo / d.da, row_hi = hi / d.da;  // steps along a, counted through the dimensions slower than it
  const uint64_t at_lo = row_lo / d.ea * d.tiles_a + row_lo % d.ea / d.ta;
  const uint64_t at_hi = row_hi / d.ea * d.tiles_a + row_hi % d.ea / d.ta;
  *first = at_lo * group;
  *last = (at_hi + 1) * group;
  if (row_lo == row_hi && group == d.tiles_b) {  // inside one row: a block's units (lines) can reach into the next block
    const uint64_t bytes = (uint64_t)d.tb * d.run, from = lo - row_lo * d.da, reach = d.flags & kPermWide ? kPermLine - 1 : 15;
    *first += (from < reach ? 0 : from - reach) / bytes;
    *last = at_hi * group + (hi - row_hi * d.da) / bytes + 1;
  }
}
