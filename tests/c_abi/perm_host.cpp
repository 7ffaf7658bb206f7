// Host build of the block route for views with short runs (csrc/ds_perm.h, included unchanged): every block of a
// view is moved thread by thread, phase by phase, and every access is counted, so that a CPU test can see that
// exactly the bytes of the view and of the image range are read and written, and that the LDS of the kernel that runs the
// block is not left.  The gather's side of the tensor runs as in small images and as in large ones (streaming loads).
#include <stdint.h>

#include <vector>

static unsigned char *g_arena_hits, *g_image_hits;  // accesses per byte
static uint64_t g_arena, g_arena_len, g_image, g_image_len, g_lds_len;
static uint64_t g_loads, g_streamed, g_large;  // loads of the tensor: all, streaming, by the gather as in large images
static long g_bad;
static void touch(char kind, uint64_t at, uint64_t n, uint64_t align);
#define DS_PERM_TOUCH(kind, at, n, align) touch(kind, at, n, align)
#include "ds_perm.h"

static void touch(char kind, uint64_t at, uint64_t n, uint64_t align) {
  if (kind == 'l') {
    if (at + n > g_lds_len || at % align) ++g_bad;
    return;
  }
  if (kind == 'r') ++g_loads;
  if (kind == 's') ++g_loads, ++g_streamed;
  const bool arena = kind == 'r' || kind == 's' || kind == 'w';
  const uint64_t base = arena ? g_arena : g_image, len = arena ? g_arena_len : g_image_len;
  if (at < base || at + n > base + len || at % align) {
    ++g_bad;
    return;
  }
  for (uint64_t i = at - base; i < at - base + n; ++i)
    if ((arena ? g_arena_hits : g_image_hits)[i] < 255) ++(arena ? g_arena_hits : g_image_hits)[i];
}

template <typename E, typename W>
static void move_block(const DsPerm &d, const DsPermBlock &k, bool pack, unsigned char *img, uint64_t lo, uint8_t *lds) {
  const auto store = [](uint64_t p, const DsPermUnit &v) { memcpy((void *)(uintptr_t)p, v.w, 16); };
  const auto load = [](uint64_t p) {
    DsPermUnit v;
    memcpy(v.w, (const void *)(uintptr_t)p, 16);
    return v;
  };
  g_lds_len = d.flags & kPermWide ? kPermLdsBytes : kPermNarrowBytes;
  memset(lds, 0xCD, kPermLdsBytes);
  for (uint32_t t = 0; t < kPermThreads; ++t)
    if (pack) ds_perm_tensor_side<E, W, true>(d, k, lds, t);
    else ds_perm_image_load(d, k, lds, img, lo, t, load);
  if (pack) {
    alignas(16) static uint8_t streamed[kPermLdsBytes];
    memset(streamed, 0xCD, kPermLdsBytes);
    const uint64_t before = g_loads;
    for (uint32_t t = 0; t < kPermThreads; ++t) ds_perm_tensor_side<E, W, true, true>(d, k, streamed, t);
    g_large += g_loads - before;
    if (memcmp(lds, streamed, kPermLdsBytes)) ++g_bad;
  }
  for (uint32_t t = 0; t < kPermThreads; ++t)
    if (pack) ds_perm_image_store<E>(d, k, lds, img, lo, t, store);
    else ds_perm_tensor_side<E, W, false>(d, k, lds, t);
}

static uint32_t g_flags;  // of the last view
static uint64_t g_image_bytes = 1 << 20;  // the whole image's, by which the plan chooses the size of some blocks
extern "C" void perm_host_image_bytes(uint64_t n) { g_image_bytes = n; }
// The loads of the tensor by gathers as in images that no cache holds, and how many of them streamed.
extern "C" uint64_t perm_host_loads() { return g_large; }
extern "C" uint64_t perm_host_streamed() { return g_streamed; }
// Is the last view moved 16 bytes along the columns at a time?
extern "C" int perm_host_groups() { return (g_flags & kPermGroups) != 0; }
// Do the scatter's loads of the image stream for the last view?
extern "C" int perm_host_image_streams() { return (g_flags & kPermImageOnce) != 0; }

// Moves image bytes [lo, hi) of one view at image offset `at`; `img` holds byte lo.  Returns the number of blocks
// (0: not this route's), or -1 if an access was out of bounds or not aligned.  Runs the blocks that a launch for the
// range would have, which perm_host_launched counts.
static uint64_t g_launched;
extern "C" uint64_t perm_host_launched() { return g_launched; }
extern "C" long perm_host_move(unsigned char *arena, uint64_t arena_len, uint64_t offset, uint64_t at, uint64_t nbytes,
                               uint64_t run, uint32_t n_outer, const uint64_t *extent, const uint64_t *stride, int pack,
                               uint64_t lo, uint64_t hi, unsigned char *img, unsigned char *arena_hits,
                               unsigned char *image_hits) {
  g_arena = (uint64_t)(uintptr_t)arena;
  g_arena_len = arena_len;
  g_image = (uint64_t)(uintptr_t)img;
  g_image_len = hi - lo;
  g_arena_hits = arena_hits;
  g_image_hits = image_hits;
  g_bad = 0;
  alignas(16) static uint8_t lds[kPermLdsBytes];
  DsPerm d;
  const uint64_t n = ds_perm_make(g_arena + offset, at, nbytes, run, n_outer, extent, stride, g_image_bytes, &d);
  if (n) g_flags = d.flags;
  uint64_t first = 0, last = n;
  if (n) ds_perm_range(d, lo, hi, &first, &last);
  if (last > n) ++g_bad;
  std::vector<DsPermItem> items(n);
  if (n) ds_perm_items(d, 0, (uint32_t)n, items.data());
  g_launched += last - first;
  for (uint64_t t = first; t < last; ++t) {
    DsPermBlock k;
    if (!ds_perm_block(d, items[t].tile, lo, hi, pack, k)) continue;
    switch (d.flags & 0xFFu) {
      case 0: move_block<uint8_t, uint32_t>(d, k, pack, img, lo, lds); break;
      case 1: move_block<uint16_t, uint32_t>(d, k, pack, img, lo, lds); break;
      case 2: move_block<uint32_t, uint32_t>(d, k, pack, img, lo, lds); break;
      default: move_block<uint64_t, uint64_t>(d, k, pack, img, lo, lds); break;
    }
  }
  return g_bad ? -1 : (long)n;
}
