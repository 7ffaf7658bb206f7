// Internal definitions shared by the host side and the kernels of
// libdatastates_hip.so.  Not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "datastates.h"
#include "ds_perm.h"

// A tile is one non-empty shard in device form: the view is normalised to
// "outer index -> start of a contiguous run of run_bytes".  Its place in the
// image is [tile_off[t], tile_off[t+1]): payload first, then padding.
struct DsTile {
  uint64_t src;        // device address of element (0,...,0)
  uint64_t nbytes;     // payload bytes
  uint64_t run_bytes;  // length of the innermost contiguous run; == nbytes when n_outer == 0
  uint32_t n_outer;    // outer dimensions left after merging; 0 = the whole shard is one run
  uint32_t es_log2;    // log2(itemsize)
  uint64_t extent[DS_MAX_DIMS];  // outer extents, slowest first
  uint64_t stride[DS_MAX_DIMS];  // outer strides in BYTES
};
static_assert(sizeof(DsTile) == 128, "DsTile is one 128-byte line");

// What the kernel's general path needs of a tile, 40 bytes instead of the 128 of a DsTile plus its two
// tile_off entries: the first wavefront of a general chunk reads one of these per lane.  Entry n_tiles is
// a sentinel whose img_off is the image length, so that a tile's end is the next entry's img_off.
struct DsTileHot {
  uint64_t img_off;  // where the tile's range starts in the image (= tile_off[t])
  uint64_t src;      // device address of element (0,...,0)
  uint64_t nbytes;   // payload bytes
  uint64_t stride0;  // distance between runs in bytes (views with one outer dimension)
  uint32_t run;      // run length in bytes, views with one outer dimension (0 otherwise)
  uint32_t meta;     // n_outer | log2(itemsize) << 8 | DS_HOT_*.  n_outer is given as 2 for a view with one
                     // outer dimension whose runs do not fit 32 bits: it then takes the routes of the N-D views
};
enum : uint32_t {
  DS_HOT_PERM = 1u << 17,  // the view's whole units are moved in blocks (ds_perm.h)
  DS_HOT_LANES = 1u << 18  // a view of less than 4 GiB with runs shorter than 16 bytes, of which the general path moves so
                           // little that it does so an element per lane: what is left of a view moved in blocks, and views
                           // with runs of one element of 1 or 2 bytes, of which the plan has at most kLanesBytes
};
// Where such views keep the chip busy, the pieces of a unit one after the other are the faster way: 20 000 views of 512
// bytes (bf16, transposed) 26.5 / 32.0 us, of 400 bytes 40.0 / 45.2; 300 of them 9.2 / 7.1 and 15.9 / 11.5.  Runs of several
// elements, and elements of 4 bytes and more, have fewer pieces (300 views with rows of 9 bytes 5.5 / 6.7, every second of
// 20 floats 5.7 / 6.1).
constexpr uint64_t kLanesBytes = 256 << 10;
static_assert(sizeof(DsTileHot) == 40, "five 8-byte words");

// What the kernel's lean path needs to move one whole chunk, in one 32-byte load.
// Chunks that are not "simple" (a tile boundary, the end of a payload or
// padding inside the chunk, more than one outer dimension, rows shorter than
// 16 bytes) are of kind DS_CHUNK_GENERAL and take the general path; their
// record names the tiles they hold (tile, col0).  DS_CHUNK_PERM: the whole chunk is whole units of one view that is
// moved in blocks (ds_perm.h); its record is that of a general chunk, for launches without the block tables.
// DS_CHUNK_MULTI: general, and every tile of it is one contiguous run; same record.
// DS_CHUNK_DIMS: the whole chunk is whole units of one view with several outer dimensions, fewer than 2^32 runs of 16 bytes
// and more; the record of a general chunk, with addr = number of the run that holds the chunk's first byte, pitch = that
// byte's position in it, run.
enum : uint32_t {
  DS_CHUNK_CONTIG = 0, DS_CHUNK_ROWS = 1, DS_CHUNK_GENERAL = 2, DS_CHUNK_PERM = 3, DS_CHUNK_MULTI = 4, DS_CHUNK_DIMS = 5
};
constexpr uint32_t kMultiTiles = 1024;  // tiles a chunk of kind DS_CHUNK_MULTI may hold
// CONTIG only, bit 8 of `kind`: the tensor side of the chunk is not 16-byte aligned, and the tensor has at least
// 16 more bytes on either side of it, so the gather may read the 16-byte aligned units that cover the chunk's
// bytes (one more than the chunk has) without leaving the tensor.
enum : uint32_t { DS_CHUNK_REALIGN = 1u << 8 };
struct DsChunkRec {
  uint64_t addr;   // CONTIG: tensor address of the chunk's first byte; ROWS: address of the run that holds it
  uint64_t pitch;  // ROWS: distance between runs in bytes
  uint32_t col0;   // ROWS: position of the chunk's first byte inside its run.  GENERAL: number of tiles after the first
  uint32_t run;    // ROWS: run length in bytes (>= 16, multiple of the itemsize)
  uint32_t kind;   // low byte: DS_CHUNK_*; bits 8..: log2(itemsize) (ROWS), DS_CHUNK_REALIGN (CONTIG)
  uint32_t tile;   // GENERAL: first tile of the chunk.  ROWS: (step / run) << 16 | (step % run), step = bytes
                   // between two units of one thread (threads per work-group x 16)
};
static_assert(sizeof(DsChunkRec) == 32, "two records per 64 bytes");

struct DsManifestEntry {
  uint64_t tensor_id;
  uint32_t dtype;
  uint32_t ndim;
  int64_t shape[DS_MAX_DIMS];  // unused extents 0
  uint64_t file_offset;   // inside the shard's own file
  uint64_t nbytes;
  uint64_t image_offset;  // in the plan's image (= file_offset + where the file's region starts)
  uint32_t file;
};

// One file of a flush or of a restore: image bytes [begin, end) are the file's bytes [0, end - begin).
// fd_direct may be -1.
struct DsFileTarget {
  uint64_t begin = 0, end = 0;
  int fd_buffered = -1, fd_direct = -1;
};

// The flush of a snapshot into a file that somebody else opened and will close (the checkpoint writer).
// fd_direct may be -1.
int ds_flush_start_fds(ds_event *ev, int fd_buffered, int fd_direct, uint32_t threads, uint32_t flags, ds_flush **out);
// The same into several files: the targets are in image order, the first begins at 0 and each begins where
// the one before ends.  May throw std::bad_alloc (the vector is taken by value).
int ds_flush_start_targets(ds_event *ev, std::vector<DsFileTarget> targets, uint32_t threads, uint32_t flags,
                           ds_flush **out);
// Image -> tensors out of files that the caller opened and will close; the targets must cover the image.
int ds_restore_from_targets(ds_engine *engine, const ds_plan *plan, const std::vector<DsFileTarget> &targets,
                            uint32_t threads, void *compute_stream, ds_event **out);
const ds_plan *ds_event_plan(const ds_event *ev);  // the plan a snapshot or restore was started with
void ds_set_errno(int e);  // what ds_last_errno() returns on this thread
bool ds_io_uring_available();  // can this process set up an io_uring?
void ds_drop_pinned_cache();   // frees the pinned ring kept from a destroyed engine

struct ds_plan {
  uint64_t align = 0;
  uint64_t total_bytes = 0;
  uint64_t payload_bytes = 0;
  uint64_t n_shards = 0;
  uint64_t n_strided = 0;
  uint32_t chunk_log2 = 0;
  std::vector<DsManifestEntry> manifest;   // table order as given
  std::vector<uint64_t> file_begin;        // n_files + 1 entries: where each file's tensor region starts in the image
  std::vector<DsTile> tiles;               // image order
  std::vector<uint64_t> tile_off;          // n_tiles + 1 entries, last = total_bytes (host only)
  std::vector<DsTileHot> hot;              // n_tiles + 1 entries, image order, last = sentinel
  std::vector<uint32_t> first_tile;        // n_chunks + 1 entries, last = n_tiles
  std::vector<DsChunkRec> recs;            // one per chunk
  std::vector<DsPerm> perms;               // views moved in blocks, image order
  std::vector<DsPermItem> perm_items;      // their blocks, view by view
  std::vector<uint32_t> perm_first;        // perms.size() + 1 entries: a view's first block
  // The other chunks and their records, so that a launch of those has no empty work items: in a plan of at most
  // kListAlways chunks, or where at least one chunk in kListShare is of kind DS_CHUNK_PERM.  In a larger plan with fewer
  // of them such chunks are work items that end at their record, and the list would be nearly a second copy of the table.
  // (300 MB rank with 2.8 % such chunks: gather 102.8 to 103.2 us, with a list 102.5; a list of the 7.6 GB rank with one
  // transposed matrix of 16 KiB: plan in 25 ms on the host, without it in 3.  In short launches the empty items count:
  // 25 MB with 8 % of them 17.5 us, with a list 16.8.)
  static constexpr uint64_t kListAlways = 8192, kListShare = 16;
  bool listed = false;
  std::vector<uint32_t> rest_ids;
  std::vector<DsChunkRec> rest_recs;
  uint64_t n_general = 0;                  // chunks that are not lean (kinds DS_CHUNK_GENERAL, _PERM and _MULTI)
  uint64_t n_perm_chunks = 0;              // of these the ones of kind DS_CHUNK_PERM
  uint64_t n_multi = 0;                    // ... of kind DS_CHUNK_MULTI
  uint64_t n_dims = 0;                     // ... of kind DS_CHUNK_DIMS
  uint64_t n_one_by_one = 0;               // ... and those with (parts of) views of several outer dimensions
  uint64_t n_short_rows = 0;               // chunks of rows of at most 512 bytes
  uint64_t n_rests = 0;                    // chunks of kind DS_CHUNK_GENERAL and _MULTI, in plans with blocks
  uint64_t rest_units = 0, rest_most = 0;  // ... their units that no block moves, and the most that one of them has
  bool any_wide = false;                   // does a view of `perms` move in wide blocks (ds_perm.h)?
  uint64_t n_column_blocks = 0;            // blocks that are neither wide nor one piece of the image and go along a
  uint64_t n_far_blocks = 0;               // blocks along b that read lines which blocks far on read too
  bool all_contiguous = false;             // no chunk needs the general path: every shard is one contiguous run
  // The tables the kernels read, laid out one behind the other at these offsets (multiples of 128); the tables of
  // views moved in blocks come last.  `blob` is that layout on the host for tables of up to 256 KiB and for plans that
  // only ds_pack_noalloc can use, as far as its static table memory holds them: one copy then takes it to the device.
  // (Larger device plans do without: for the 7B rank's 3.4 MB it would be 0.13 ms more per plan.)
  struct Layout {
    size_t hot = 0, first_tile = 0, recs = 0, perms = 0, perm_items = 0, rest_ids = 0, rest_recs = 0, total = 0;
  } at;
  std::vector<uint8_t> blob;
  // device copies (one allocation)
  int device = -1;
  void *dev_blob = nullptr;
  const DsTile *d_tiles = nullptr;
  const DsTileHot *d_hot = nullptr;
  const uint32_t *d_first_tile = nullptr;
  const DsChunkRec *d_recs = nullptr;
  const DsPerm *d_perms = nullptr;
  const DsPermItem *d_perm_items = nullptr;
  const uint32_t *d_rest_ids = nullptr;
  const DsChunkRec *d_rest_recs = nullptr;
  uint64_t n_chunks() const { return first_tile.empty() ? 0 : first_tile.size() - 1; }
  // Are most chunks of a launch general?  With `blocks` the launch leaves the chunks of kind DS_CHUNK_PERM to another.
  bool mostly_general(bool blocks) const {
    const uint64_t left_out = blocks ? n_perm_chunks : 0;
    return (n_general - left_out) * 2 > n_chunks() - left_out;
  }
  // Do the chunks beside the blocks hold little else than what blocks move: at most one unit for each thread of a work-group?
  // (Three quarters of them, on average; each of them where few run at once and the launch takes as long as the slowest.)
  // See ds_mixed_kernel.
  static constexpr uint64_t kRestUnits = 256;
  bool mostly_rests(bool at_once) const {
    return n_rests * 4 > rest_recs.size() * 3 && (at_once ? rest_most <= kRestUnits : rest_units <= n_rests * kRestUnits);
  }
  // Are most blocks narrow ones along a, or along b with lines that others far on read too (see ds_perm_order)?
  bool mostly_columns() const { return n_column_blocks * 2 > perm_items.size(); }
  bool mostly_far() const { return n_far_blocks * 2 > perm_items.size(); }
  // Do most chunks of a launch hold several contiguous tensors, in a plan that has views too and an image of more than
  // 16 MiB?  They then take the general path with four units per thread, whose chain of dependent loads (record,
  // descriptors, data) one unit per thread, with a quarter of the bytes in flight, pays four times.  Four units / one, us,
  // gather and scatter, tensors of one size beside a small view: 100 MB of 4 KiB 42.3 / 48.4 and 41.4 / 46.1, 48 MB of
  // 20 KB, out of the last-level cache, 21.8 / 24.3 and 22.4 / 24.5, in it 16.6 / 17.8 and 17.5 / 18.5, 36 MB of 300 bytes
  // 15.9 / 17.7 and 16.4 / 16.7; 16 MB 9.0 / 9.1 and 9.0 / 9.1; 4 MB of 4 KiB 5.1 / 3.8 and 6.4 / 4.1.  Not where the chunks hold views: 20
  // MB of 60 000 fragments, a third of them rows, 27.4 / 26.2 and 25.8 / 23.4, of rows only 37.1 / 31.5 and 34.0 / 28.5.
  bool mostly_several(bool blocks) const {
    const uint64_t left_out = blocks ? n_perm_chunks : 0;
    return !all_contiguous && total_bytes > (16ull << 20) && n_multi * 2 > n_chunks() - left_out;
  }
  // Is a scatter of `chunks` whole chunks of 16 KiB by ds_move_kernel launched in pieces of 8 KiB, six wavefronts per
  // SIMD instead of four?  (Images of 64 GiB and more, and the options for comparison: every other default call
  // launches ds_unit_kernel, which takes 4 KiB at eight.)  Measured over tables of one kind, pieces / whole, us.
  // Many rounds: pieces (7B rank 490 / 504).  Fewer chunks than give each CU two work-groups: pieces (383 chunks of rows of 1000 bytes 6.2 / 7.2, one tensor 4.3 / 4.3).
  // Between them, by what the chunks hold:
  //   one in sixteen or more views of several outer dimensions, whose units move one by one: pieces at any size (443
  //     chunks 7.4 / 9.3, 1082 13.0 / 15.6, 4889 33.7 / 36.2);
  //   one in five or more rows of at most 512 bytes: whole while all chunks run at once (926 chunks 8.8 / 7.9, 700
  //     6.7 / 6.0), and beyond that pieces where their last round is the fuller one (1405 chunks, 1.4 rounds of 1024
  //     against 1.8 of 1536: 10.9 / 11.3);
  //   anything else: whole up to two rounds (700 chunks of tensors of 300 KB 7.1 / 6.6, 900 of rows of 3000 bytes 9.4 /
  //     8.0, 1200 of one tensor 8.8 / 8.3, 1800 of rows 15.2 / 14.0), then by the rounds too (2200 chunks 15.1 / 15.2,
  //     3072 19.2 / 19.5, 2402 16.2 / 15.7).
  bool scatter_in_pieces(uint64_t chunks) const {
    if (chunks <= 384 || chunks > 8 * 1024 || n_one_by_one * 16 >= n_chunks()) return true;
    if (chunks <= (n_short_rows * 5 >= n_chunks() ? 1024u : 2048u)) return false;
    const uint64_t whole = (chunks + 1023) / 1024 * 1024, pieces = (2 * chunks + 1535) / 1536 * 768;
    return pieces * 21 <= whole * 20;
  }
};

// Copies the plan's tables in their layout to dst_dev on `stream`, the block tables if `blocks`.
int ds_copy_tables(const ds_plan *plan, bool blocks, uint8_t *dst_dev, hipStream_t stream);

// ---- error plumbing ---------------------------------------------------------
void ds_set_hip_error(hipError_t e);
#define DS_HIP_TRY(expr)                 \
  do {                                   \
    hipError_t _e = (expr);              \
    if (_e != hipSuccess) {              \
      ds_set_hip_error(_e);              \
      return DS_EHIP;                    \
    }                                    \
  } while (0)

// ---- tunables ---------------------------------------------------------------
uint64_t ds_cfg_chunk_bytes();
uint64_t ds_cfg_variant();

// ---- kernel launchers (ds_kernels.hip) ---------------------------------------
// Moves image bytes [img_lo, img_hi) between the tensors of `plan` and `img`
// (which points at image byte img_lo).  pack: tensors -> img; else img -> tensors.
// grid_limit 0 = one work-group per chunk.
int ds_launch_move(const ds_plan *plan, bool pack, uint8_t *img, uint64_t img_lo, uint64_t img_hi,
                   uint32_t grid_limit, hipStream_t stream);
