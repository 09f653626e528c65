// Types shared by the host side of the library and its kernels (not part of the C ABI).
#pragma once

#include <cstdint>
#include <vector>

#include "noloco.h"

namespace noloco {

constexpr int kBlockThreads = 256;   // four wave64 per workgroup (replica spread, probes)
constexpr int kVecElems = 4;         // one 16-byte fp32 vector per lane and load
constexpr int kStepThreads = 64;     // the outer step: one wave per workgroup ...
constexpr int kPieceElems = kStepThreads * kVecElems;   // ... which covers one piece of a tile
constexpr int kLdsBytes = 160 * 1024;   // LDS of a CU, handed out in units of kLdsUnit
constexpr int kLdsUnit = 1280;
constexpr int64_t kCus = 256;           // MI355X
constexpr int kSpreadColumns = 1024;    // columns that a workgroup of the replica-spread pass takes at a time

// A maximal contiguous run of arena elements, cut into tiles of `tile_elems` columns whose
// boundaries sit at multiples of tile_elems in row coordinates.  The run's first and last
// tile may be partial; all others are whole.
struct Span {
  int64_t col_begin;     // first element of the run (inclusive)
  int64_t col_end;       // one past its last element
  int64_t first_block;   // col_begin / tile_elems
  int64_t tile_prefix;   // number of tiles in all earlier spans
};

#if defined(__HIP__)
#define NOLOCO_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define NOLOCO_HOST_DEVICE inline
#endif

// The piece of a row that a workgroup (one wave) works on, and for which group.
struct Piece {
  uint32_t group;
  int64_t base;      // first column of the piece, a multiple of kPieceElems
  int32_t lo, hi;    // the run owns columns [base + lo, base + hi) of it, 0 <= lo < hi <= kPieceElems
  NOLOCO_HOST_DEVICE bool whole() const { return lo == 0 && hi == kPieceElems; }
};

// Which columns of the piece at r.base the run owns; false if none.
NOLOCO_HOST_DEVICE bool cut_to_run(int64_t run_begin, int64_t run_end, Piece& r, int32_t elems = kPieceElems) {
  const int64_t lo = run_begin - r.base, hi = run_end - r.base;
  r.lo = lo > 0 ? (lo < elems ? static_cast<int32_t>(lo) : elems) : 0;
  r.hi = hi < elems ? (hi > 0 ? static_cast<int32_t>(hi) : 0) : elems;
  return r.lo < r.hi;
}

// Which piece workgroup `block` of an in-order launch takes.  The hardware deals workgroups to the 8 XCDs
// in turn.  xcd_run = 1: as dealt.  xcd_run = 0: nearly so, but every other eight pieces swap their halves, so that an XCD
// meets odd and even 4 KiB pages alike (its L2 spreads them over its channels).  Otherwise each XCD takes
// runs of xcd_run pieces.  A permutation of every in_order_round(xcd_run) consecutive workgroups.
NOLOCO_HOST_DEVICE uint32_t in_order_swap(uint32_t xcd_run) { return xcd_run == 0 ? 4u : 0u; }
NOLOCO_HOST_DEVICE uint32_t piece_of_block(uint32_t block, uint32_t xcd_run, uint32_t swap) {
  if (__builtin_expect(xcd_run <= 1, 1)) return block ^ ((block >> 1) & swap);
  const uint32_t xcd = block & 7u, slot = block >> 3, k = slot / xcd_run;
  return (k * 8 + xcd) * xcd_run + (slot - k * xcd_run);
}
NOLOCO_HOST_DEVICE uint32_t in_order_round(uint32_t xcd_run) { return 8 * (xcd_run == 0 ? 1 : xcd_run); }

// What a workgroup of an arena of several runs needs to know of a cell of 2^cell_shift tiles: the cell's first two
// spans, and which spans its other tiles lie in.  Tiles are counted from the cell's first one ("at"), in 32 bits, so
// that the whole look-up is a load of one line and a few scalar instructions.
struct alignas(64) SpanCell {
  int64_t block[2];        // the tile at `at` is block at + block[i] of the row in the i-th span
  uint32_t end_at[2];      // where the i-th span ends (the next one begins), possibly beyond the cell
  uint32_t begin_col[2];   // columns from begin_col on of its first tile are the run's: 0 if it begins before the cell
  uint32_t end_col[2];     // columns [0, end_col) of its last tile are the run's
  int32_t span, last_span; // spans of the cell's first and last tile
};

// Tile `tile` of a table whose tiles have `elems` columns: its cell holds the two spans that most cells have; where
// more runs begin inside the cell (hundreds, where one run is much longer than the others, since the cells are sized
// by the mean run), a binary search over the others follows.  (The pointer types differ between host and device.)
template <typename CellPtr, typename SpanPtr>
NOLOCO_HOST_DEVICE bool locate_by_cells(CellPtr cells, int32_t cell_shift, SpanPtr spans, int64_t tile, Piece& r, int32_t elems = kPieceElems) {
  const CellPtr cell = cells + (tile >> cell_shift);
  const uint32_t at = static_cast<uint32_t>(tile) & ((1u << cell_shift) - 1u);
  const int64_t block[2] = {cell->block[0], cell->block[1]};
  const uint32_t end_at[2] = {cell->end_at[0], cell->end_at[1]}, begin_col[2] = {cell->begin_col[0], cell->begin_col[1]};
  const uint32_t end_col[2] = {cell->end_col[0], cell->end_col[1]};
#if defined(__HIP_DEVICE_COMPILE__)
  // The whole line in one round trip: otherwise the compiler loads the ends first, and the rest after the branch.
  asm volatile("" :: "s"(block[0]), "s"(block[1]), "s"(end_at[0]), "s"(end_at[1]), "s"(begin_col[0]), "s"(begin_col[1]),
               "s"(end_col[0]), "s"(end_col[1]));
#endif
  const int second = at >= end_at[0] ? 1 : 0;
  if (at < end_at[1]) {
    r.base = ((second ? block[1] : block[0]) + static_cast<int64_t>(at)) * elems;
    r.lo = at == (second ? end_at[0] : 0u) ? static_cast<int32_t>(second ? begin_col[1] : begin_col[0]) : 0;
    r.hi = at + 1u == (second ? end_at[1] : end_at[0]) ? static_cast<int32_t>(second ? end_col[1] : end_col[0]) : elems;
    return true;
  }
  int32_t lo = cell->span + 2, hi = cell->last_span + 1;
  while (hi - lo > 1) {
    const int32_t mid = lo + (hi - lo) / 2;
    if (spans[mid].tile_prefix <= tile) lo = mid; else hi = mid;
  }
  r.base = (tile + spans[lo].first_block - spans[lo].tile_prefix) * elems;
  return cut_to_run(spans[lo].col_begin, spans[lo].col_end, r, elems);
}

// Piece `piece` of tile `tile` of any table, by binary search.
template <typename SpanPtr>
NOLOCO_HOST_DEVICE bool locate_by_search(SpanPtr spans, int32_t num_spans, int32_t piece_shift, int64_t tile,
                                         uint32_t piece, Piece& r) {
  int lo = 0, hi = num_spans;               // spans[hi] is the sentinel: its prefix is the tile total
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (spans[mid].tile_prefix <= tile) lo = mid; else hi = mid;
  }
  r.base = (((spans[lo].first_block + (tile - spans[lo].tile_prefix)) << piece_shift) + piece) * kPieceElems;
  return cut_to_run(spans[lo].col_begin, spans[lo].col_end, r);
}

// How an in-order launch of groups of up to 16, or in phases, stores whole pieces: with non-temporal stores, written through the L2, or
// through the L2 but kept in the memory's cache.
enum Stores : uint32_t { kStreaming, kThrough, kKept };

// A launch in phases: the whole chip reads for half a period and writes for the other half, see phases_of_launch().
struct Phases {
  uint32_t per_tick;       // 2^32 over the period in ticks of the GPU's constant clock; 0 = no phases
  uint32_t class_shift;    // workgroups are dealt, kCus at a time, to 2^class_shift classes, as many as a CU holds waves
  uint32_t store_for;      // how long after the beginning of a class's part its stores may begin, in 2^-32 of the period
  uint32_t width;          // workgroups per group of the launch, and all of it (set for the launch)
  uint32_t workgroups;
};
constexpr int32_t kPhasedLeast = 2, kPhasedMost = 56;      // sizes of groups that have such launches
// Time within the period, in 2^-32 of it: reads in the first half, each class's stores in its part of the second.
constexpr uint32_t kHalfPeriod = 0x80000000u;
NOLOCO_HOST_DEVICE uint32_t phase_round(uint32_t class_shift) { return static_cast<uint32_t>(kCus) << class_shift; }
NOLOCO_HOST_DEVICE uint32_t store_phase(uint32_t workgroup, uint32_t class_shift) {
  return kHalfPeriod + (workgroup / static_cast<uint32_t>(kCus) & ((1u << class_shift) - 1u)) * (kHalfPeriod >> class_shift);
}

// Kernel arguments of one launch: all groups in it have the same size n.
struct StepArgs {
  float* phi;
  float* delta;
  void* theta;
  int64_t stride;          // elements between rows
  int64_t run_begin;       // an arena of one run: its columns [run_begin, run_end), and
  int64_t run_end;
  int64_t first_piece;     // the piece that its first tile begins with (set for the launch from tile_offset)
  const Span* spans;       // device, num_spans + 1 entries (last is a sentinel holding the tile total)
  const SpanCell* cells;   // device, more than one run: cell of tile t at t >> cell_shift; else null
  int32_t cell_shift;
  uint32_t num_pieces;     // in order: pieces of the launch, see piece_of_block() (set for the launch)
  uint32_t xcd_run;
  uint32_t stores;         // Stores, of whole pieces in launches in order
  float alpha, beta, gamma, inv_n;
  int32_t n;               // group size
  int64_t tile_offset;     // first of the launch's tiles: it covers [tile_offset, tile_offset + num_tiles)
  int64_t num_tiles;       // tiles per group taken by this launch
  int32_t num_groups;      // groups in this launch
  int32_t num_spans;
  int32_t piece_shift;     // a tile is 2^piece_shift pieces, one workgroup each
  int32_t group_major;     // work item -> (tile, group) order
  int32_t xcd_map;         // workgroup -> work item permutation, see noloco_tuning
  uint32_t work_items;     // num_tiles * num_groups
  Phases phases;           // in order
  int32_t rows[NOLOCO_MAX_GROUP];  // group g = rows[g*n .. g*n+n), ascending worker ids
};

// How the workgroups of an in-order launch find their pieces.
struct InOrderHead {
  const SpanCell* cells;   // several runs
  const Span* spans;
  int64_t first;           // several runs: the launch's first tile; one run: the first piece of the row that the launch owns
  uint32_t num_pieces;
  uint32_t xcd_run;        // see piece_of_block()
  uint32_t swap;           // in_order_swap(xcd_run)
  uint32_t cell_shift;
  uint32_t begin_col;      // one run: columns [begin_col, kPieceElems) of the first piece are the run's,
  uint32_t end_col;        // and columns [0, end_col) of the last
};

// host: the head of a launch as part_of_launch() cut it
inline InOrderHead in_order_head(const StepArgs& a) {
  InOrderHead h = {a.cells, a.spans, a.tile_offset, a.num_pieces, a.xcd_run, in_order_swap(a.xcd_run),
                   static_cast<uint32_t>(a.cell_shift), 0, kPieceElems};
  if (a.cells == nullptr) {
    const int64_t begin = a.run_begin / kPieceElems, end = (a.run_end - 1) / kPieceElems, beyond = a.first_piece + a.num_pieces;
    h.first = a.first_piece > begin ? a.first_piece : begin;
    h.begin_col = h.first == begin ? static_cast<uint32_t>(a.run_begin % kPieceElems) : 0u;
    h.end_col = end < beyond ? static_cast<uint32_t>((a.run_end - 1) % kPieceElems) + 1u : static_cast<uint32_t>(kPieceElems);
    h.num_pieces = static_cast<uint32_t>((end < beyond ? end + 1 : beyond) - h.first);
  }
  return h;
}

// Workgroup `block` of an in-order launch -> its piece.  An arena of one run takes no load but that of the arguments;
// with more runs the table of cells usually costs one more.  (CellPtr and SpanPtr convert from the pointers in the
// head.)
template <typename CellPtr, typename SpanPtr>
NOLOCO_HOST_DEVICE bool locate_by_head(const InOrderHead& h, uint32_t block, Piece& r) {
  const uint32_t piece = piece_of_block(block, h.xcd_run, h.swap);
  if (piece >= h.num_pieces) return false;
  if (h.cells == nullptr) {
    r.base = (h.first + static_cast<int64_t>(piece)) * kPieceElems;
    r.lo = piece == 0 ? static_cast<int32_t>(h.begin_col) : 0;
    r.hi = piece + 1 == h.num_pieces ? static_cast<int32_t>(h.end_col) : kPieceElems;
    return true;
  }
  return locate_by_cells((CellPtr)(h.cells), static_cast<int32_t>(h.cell_shift), (SpanPtr)(h.spans), h.first + static_cast<int64_t>(piece), r);
}
template <typename CellPtr, typename SpanPtr>
bool locate_in_order(const StepArgs& a, uint32_t block, uint32_t group, Piece& r) {
  r.group = group;
  return locate_by_head<CellPtr, SpanPtr>(in_order_head(a), block, r);
}

// Which tile workgroup `block` of the replica-spread pass takes: each XCD takes runs of 2^run_shift.
NOLOCO_HOST_DEVICE uint32_t tile_of_block(uint32_t block, uint32_t run_shift) {
  const uint32_t xcd = block & 7u, slot = block >> 3;
  return ((((slot >> run_shift) << 3) + xcd) << run_shift) + (slot & ((1u << run_shift) - 1u));
}

// One workgroup's share of pooling the tile sums.
struct PoolJob {
  enum Kind : int32_t {
    kChunk,        // `count` tile sums from `first` on, a part of a tensor that has several chunks
    kWhole,        // tensor `first`, by the whole workgroup
    kBatch,        // the tensors [first, first + count) of at most kPoolChunk tiles
    kShortBatch    // those of them of at most kPoolShort tiles: the longer ones have jobs of their own
  };
  int64_t first;
  int32_t count;
  Kind kind;
};

// Tensors with more tiles than this are pooled in chunks of it (eight loads per thread of a workgroup).
constexpr int64_t kPoolChunk = 2048;
// Tensors of a batch: kPoolLanes lanes each, as many loads per lane; a longer one is pooled by a wave.
constexpr int kPoolLanes = 8;
constexpr int64_t kPoolShort = kPoolLanes * kPoolLanes;
constexpr int64_t kPoolSegments = kBlockThreads / kPoolLanes;   // tensors a workgroup takes at a time

// Kernel arguments of the replica-spread pass (one tile = tile_elems columns of ONE tensor).
struct SpreadArgs {
  const void* x;           // [W][stride] float or bf16
  int64_t stride;
  const SpanCell* cells;   // over the spans' tiles
  const Span* spans;       // one span per non-empty segment, caller's order, + sentinel
  int32_t cell_shift;
  int32_t W;
  float inv_W;
  uint32_t tiles;
  uint32_t run_shift;      // each XCD takes runs of 2^run_shift tiles
  int32_t tile_elems;      // kSpreadColumns, or four times that
  double* partials;        // [tiles] sum over the tile's owned columns of the per-column variance,
                           // then [segments] sums per tensor, then the ticket
  const PoolJob* jobs;     // device
  const int32_t* long_segments;  // device: the segments that are pooled in chunks
  int32_t num_jobs;
  int32_t num_long;
  uint32_t* ticket;        // workgroups of the pooling kernel that have ended
  double elements;         // of all segments
};

// One entry per segment in the caller's order (empty ones included): where its tiles' partial
// sums sit and how many elements it has.
struct SegmentTiles {
  int64_t first_tile;
  int64_t num_tiles;
  int64_t numel;
};

// Groups of different sizes up to 16 that share an in-order launch, gathered size by size.
constexpr int32_t kMixedRows = 64;
struct Together {
  int32_t groups, rows, most;            // so far, and the largest size
  int32_t usual;                         // members in groups of the size that most of them are in: the launch is paced like one of it
  uint32_t lds;
  uint32_t group[kMixedRows];            // where a group's members begin in `member`, and its size in the upper half
  int32_t member[kMixedRows];
};

struct KernelChoice {
  int32_t vectors_per_thread;
  int32_t nontemporal;
  int32_t group_major;
  int32_t xcd_map;
  int32_t in_order;        // no knob is set: pieces in the order of the arena, group by group
  uint32_t lds;            // in order: bytes of LDS that a workgroup claims to pace the launch, 0 = not paced
  Together* together = nullptr;    // in order: the groups wait there until the last size's
  bool last = false;
};

constexpr uint32_t kXcds = 8;        // MI355X: 8 accelerator dies, workgroups are dealt to them round-robin

// The HIP runtime refuses a launch whose grid.x * block.x exceeds 2^32 - 1.  Launches are cut
// (over groups and over tile ranges) so that a grid stays at or below this many workgroups;
// the margin leaves room for the rounding the XCD maps add.
constexpr int64_t kMaxGridWorkgroups = (0xFFFFFFFFll / kBlockThreads) - 8 * 4096;

// Capacity, in doubles, of the file-scope device array that noloco_replica_spread_noalloc uses
// in place of the plan's own partial-sum buffer (16 MiB per GPU).
constexpr int64_t kSpreadScratchDoubles = 2 * 1024 * 1024;

// host: segment table -> runs (sorted, merged); see noloco_merge_segments
noloco_status merge_segments(const noloco_segment* segments, int32_t num_segments,
                             int64_t worker_stride, std::vector<noloco_segment>* runs);

// host: runs -> spans for a tile size; returns the tile total
int64_t build_spans(const std::vector<noloco_segment>& runs, int32_t tile_elems,
                    std::vector<Span>* spans);

// host: cells of 2^*shift tiles over a span table, one or two of them per span
void build_cells(const std::vector<Span>& spans, std::vector<SpanCell>* cells, int32_t* shift, int32_t tile_elems = kPieceElems);

// host: how the pooling kernel shares out the tile sums of the segments
void build_pool_jobs(const std::vector<SegmentTiles>& segments, std::vector<PoolJob>* jobs,
                     std::vector<int32_t>* long_segments);

// host: waves that a CU holds of an in-order launch of `pieces` pieces which own `columns` columns of groups
// of n, 0 = as many as fit; and the LDS that each claims for that.  `apart`: the arena is so large that its arrays lie
// in different thirds of the memory; `near`: they lie next to each other.
int32_t waves_per_cu(int32_t n, bool bf16, int64_t pieces, int64_t columns, bool apart, bool near = false);
uint32_t lds_for_waves(int32_t waves);

// host: the phases of an in-order launch of groups of n whose whole pieces are written through; per_tick = 0: none.
// `near` as above.
struct LaunchColumns {
  int64_t tiles;           // pieces of a group, and the columns that its runs own of them
  int64_t columns;
  int64_t runs;
  int64_t groups;
  int64_t stride;          // elements between rows
};
Phases phases_of_launch(int32_t n, bool bf16, const LaunchColumns& c, bool near);

// host: tiles of the runs that each XCD takes of the replica-spread pass, as a power of two
uint32_t spread_run_shift(int32_t W, bool bf16, int64_t tiles, int32_t tile_elems);

// host: workgroups that a CU holds of the replica-spread pass over `tiles` tiles of `tile_elems` columns x W rows, of which
// the tensors own `columns`, 0 = as many as fit
int32_t spread_workgroups_per_cu(int32_t W, bool bf16, int64_t tiles, int64_t columns, int32_t tile_elems);

// host: the part of a launch that begins with its tile `first` (counted from args.tile_offset) and fits one
// grid; returns how many tiles that are
int64_t part_of_launch(const StepArgs& args, int64_t first, StepArgs* part);

// kernels.hip: enqueue one launch, or with choice.together none but the last size's.  Returns hipError_t as int.
int launch_outer_step(const StepArgs& args, int32_t theta_dtype, const KernelChoice& choice,
                      void* stream);
// mode 0 copy, 1 read only (dst = 4-byte sink), 2 fill
int launch_stream_probe(int mode, void* dst, const void* src, int64_t bytes, float value, void* stream);

int launch_replica_spread(const SpreadArgs& args, int32_t x_dtype, const SegmentTiles* seg_tiles,
                          int32_t num_segments, double* out_std, void* stream);

// kernels.hip: address of the current device's copy of the static scratch array (resolved once
// per device and cached).  Returns hipError_t as int; performs no allocation of its own.
int static_spread_scratch(double** out);

// tile size in elements for a kernel choice and group size
int32_t tile_elems_for(int32_t n, int32_t vectors_per_thread);
// largest tile size of the replica-spread pass for W rows: the one its size limit is stated in
int32_t spread_tile_elems_for(int32_t W);

}  // namespace noloco
