// C ABI of the NoLoCo outer step: argument checking, the launch plan, and the split of one
// outer step into kernel launches.  All arithmetic of the method is in kernels.hip.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <memory>
#include <new>
#include <vector>

#include "noloco_internal.h"

namespace {

using noloco::Span;

constexpr int32_t kTileSizes[4] = {1024, 2048, 4096, noloco::kPieceElems};
constexpr int32_t kFineTile = 3;
// From this state on (all its rows of phi, delta and theta: one third of the memory) a launch of groups of four and more gives each XCD runs of
// kApartRun pieces, 64 KiB of a row, which fill all 16 channels of its L2 whatever the rows' distance.
// 1.6 G columns x 16 bf16 rows, 258 GB, as dealt / in runs: n = 16 5692 / 6267 GB/s, n = 4 6350 / 6391,
// n = 2 6396 / 6324.  Smaller arenas next to each other: n = 16 5557 / 5239, n = 4 6154 / 5462.
constexpr int64_t kApartBytes = 96ll << 30;
constexpr uint32_t kApartRun = 64;
// Arrays whose bases are this far from each other lie in different thirds of the memory, or nearly so (a caller who
// carves them out of one block places them like that).  Closer ones are taken as next to each other, which wants
// fewer waves (see paced_waves()) and the pieces as dealt: 124 M columns x 16 float rows, halves swapped / as dealt,
// GB/s: n = 2 6515 / 6564  n = 4 6289 / 6365  n = 8 5755 / 5838  n = 16 5411 / 5521; bf16 n = 2 6680 / 6664  n = 12 5630 /
// 5756  n = 16 5481 / 5561.  Far apart n = 2 6566 / 6544  n = 8 6488 / 6473  n = 16 6311 / 6236.
// (Virtual addresses are a guess at where memory lies; an arena taken for the other kind loses 0 to 3 %.)
constexpr uint64_t kFarBytes = 64ull << 30;
// Launches in phases take them for far apart from here on: three bases half a third from each other never lie in one third.  As if
// next to each other / as if far apart, 12 GB, GB/s, bases 48 to 63 GiB from each other wherever the first lies: n = 2 float 6540 /
// 6640  n = 8 6430 / 6610, bf16 6340 / 6580  n = 16 6250 / 6525, 6090 / 6370  n = 24 bf16 6050 / 6370  n = 32 5757 / 5990 to 6190 (paced)
// n = 48 6050 / 6357, 5765 / 5880 to 6190 (paced).  Launches too short for the phases of arrays far apart are paced: 1.2 GB, n = 32
// bf16 5550 / 6070, n = 12 float 5900 / 5540.  At 24 GiB and next to each other it loses where all three lie in one third (n = 8 float
// 6410 / 6459, bf16 6323 / 6096  n = 16 6226 / 5995, 6090 / 5750  n = 48 6043 / 5535, 5748 / 5079); in between, arrays that lie in two
// thirds lose by being taken for neighbours, from 16 bf16 members on up to 4 %, from 25 on up to 7.
constexpr uint64_t kThirdsBytes = 48ull << 30;
// The results of an arena whose state is at most this stay in the 256 MB cache in front of HBM (stores without nt),
// where the inner phase that follows finds the fast weights, and the next step what that has left of the rest.  Part of
// them is written to HBM later, by whoever evicts them.  us that a step costs a training loop over one arena (W = 4, n = 2,
// float; an inner phase that reads theta twice, writes gradients, updates theta and two moments of its size and writes
// and reads activations of 64 / 256 / 1000 MB; the loop without the step taken off; +-1), results through / kept:
//   16 MB of state 7.3 / 6.2  7.1 / 7.2  6.7 / 5.6     25 MB 9.9 / 8.3  9.9 / 9.9  9.4 / 9.6     50 MB 18.2 / 15.6  19.0 / 19.6  18.0 / 17.0
//   64 MB          21.8 / 19.5  21.9 / 22.7  22.2 / 20.7    100 MB 32.5 / 29.7  32.2 / 33.6  30.1 / 33.1    160 MB 48.7 / 49.0  49.5 / 50.7  49.4 / 47.7
// so it pays where the inner phase fits the cache too, and from 100 MB on it costs as much where that does not.  bf16 and n = 1, 4
// and 16 are alike.  Steps one after the other gain more, 50 MB 18.8 / 13.3; arenas in no cache lose, n = 2 16 MB 8.2 / 8.4, 30 MB
// 12.6 / 13.2 (non-temporal 12.8), n = 1 11.4 / 12.0 (11.5), n = 4 12.6 / 13.2 (12.6), n = 2 50 MB 18.4 / 18.7.
constexpr int64_t kKeptBytes = 64ll << 20;
// Runs so short that many pieces are owned in part gain nothing from either.  What is kept goes by the mean run; what is
// written through by how many of the columns lie in runs of kLongRun and more: runs of one length lose up to 6000 columns
// and gain from 12 000 on; where lengths differ widely the long ones carry most of the columns.  Non-temporal / written
// through, in no cache, n = 2 (n = 8), float, us:
//   250 MB, runs of 0.5 to 1.5 times 3000 86.7 / 88.2 (90.5 / 90.9)  6000 84.8 / 85.3 (92.8 / 92.5)  12 000 83.1 / 82.4 (90.6 / 89.4)
//   5 GB                                1730 / 1763 (1925 / 1959)      1717 / 1726 (1868 / 1916)      1686 / 1637 (1805 / 1817)
//   250 MB, lengths over 14 binary orders, mean 1500 (44 % of the columns in long runs) 89.9 / 91.2 (94.8 / 94.8)
//     3000 (71 %) 85.4 / 85.0 (89.5 / 87.4)  6000 (85 %) 82.9 / 81.4 (87.5 / 85.3);  5 GB 1827 / 1835  1743 / 1729  1631 / 1623
// and the same within 2 % for n = 1 and 4, bf16 and 768 MB.
constexpr int64_t kKeptRun = 16384;                    // columns of the mean run
constexpr int64_t kLongRun = 8192;
// Two rows take tiles of 4096 columns from so many of them on, if the tensors fill five eighths of them.  us, 1024 / 4096
// columns: 400 MB in 16 384 tensors, bf16 (60 % full) 83.4 / 89.2, float (43 %) 84.0 / 82.6, in 65 536 bf16 (27 %) 150 / 205, float 148 / 187;
// 4 GB in 65 536 float (65 %) 653 / 640, bf16 (79 %) 671 / 640, in one tensor float 570 / 566, bf16 567 / 549; fewer tiles, 100 MB in one
// tensor, 21.8 / 21.8 and 22.1 / 21.3.
constexpr int64_t kSpreadPairTiles = 8192;
// Groups of different sizes share a launch up to this much of their members' state: of up to eight members, none with less
// than two nor with more than twice another's, 1 GB, from five on 400 MB; others, which a launch cannot pace alike, 32 MB.
// us, a launch for each size / one, arenas in no cache (1 MB: the host's time):
//   2 2 3 float 1 MB 8.4 / 5.1  40 MB 18.4 / 16.5  200 MB 67.0 / 64.9  800 MB 257.6 / 253.5  1.6 GB 482.2 / 481.6 (bf16 491.4 / 494.2)
//   4 4 7 bf16 40 MB 18.7 / 17.7  200 MB 73.4 / 68.3  400 MB 137.6 / 133.1   5 6 7 bf16 1 MB 13.7 / 5.1  200 MB 77.6 / 69.3
//   1 2 float 40 MB 18.3 / 16.7  200 MB 64.3 / 65.5  800 MB 249.8 / 257.8
//   8 8 15 float 10 MB 10.5 / 6.9  40 MB 17.4 / 17.6  200 MB 73.8 / 68.5, bf16 100 MB 37.7 / 40.2
//   1 3 16 float 40 MB 19.5 / 16.5  100 MB 40.8 / 41.7  400 MB 149.0 / 161.9
int64_t mixed_bytes(int32_t least, int32_t most) {
  if (least < 2 || most > 8 || most > 2 * least) return 32ll << 20;
  return most <= 4 ? 1ll << 30 : 400ll << 20;
}
constexpr int64_t kFill = 256 * 8;                     // workgroups that give every CU eight

// Launch shape for subgroup size n.  With no knob set the pieces go out in the order of the arena, group
// by group, in one launch per size, paced if the launch is large.  Under explicit knobs those not given
// take the values below: pairs walk big tiles group by group; larger subgroups have smaller tiles, which
// want each XCD on a contiguous range (all 16 of its L2 channels busy) and all groups in flight at once.
noloco::KernelChoice resolve(const noloco::KernelChoice& asked, int32_t n, int64_t big_tiles) {
  noloco::KernelChoice c = asked;
  c.in_order = c.vectors_per_thread == -1 && c.nontemporal != 0 && c.group_major == -1 && c.xcd_map == -1 ? 1 : 0;
  c.lds = 0;
  if (c.vectors_per_thread == -1) {
    // `big_tiles` = workgroups the launch would have with 4096-column tiles.  An arena too small
    // to give every CU eight of them takes smaller ones, so that the maps have more to deal out.
    c.vectors_per_thread = big_tiles >= kFill ? 4 : (2 * big_tiles >= kFill ? 2 : 1);
  }
  if (c.nontemporal == -1) c.nontemporal = 1;
  if (c.group_major == -1) c.group_major = n <= 2 ? 1 : 0;
  if (c.xcd_map == -1) c.xcd_map = n <= 2 ? 0 : 1;
  return c;
}

bool aligned(const void* p, uintptr_t bytes) {
  return (reinterpret_cast<uintptr_t>(p) % bytes) == 0;
}

// Do the byte ranges [a, a + a_bytes) and [b, b + b_bytes) share a byte?
bool overlap(const void* a, uint64_t a_bytes, const void* b, uint64_t b_bytes) {
  const uintptr_t a0 = reinterpret_cast<uintptr_t>(a), b0 = reinterpret_cast<uintptr_t>(b);
  return a0 < b0 + b_bytes && b0 < a0 + a_bytes;
}

uint64_t distance(const void* a, const void* b) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x > y ? x - y : y - x;
}

}  // namespace

struct noloco_launch_plan {
  int device = -1;
  int32_t W = 0;
  int32_t theta_dtype = 0;
  int64_t stride = 0;
  int64_t elements = 0;                      // real elements per worker
  int64_t long_elements = 0;                 // those of them in runs of kLongRun and more
  std::vector<noloco_segment> runs;          // host copy, sorted and merged
  Span* dev_spans = nullptr;                 // one allocation holding all tables
  Span* dev_tables[4] = {};                  // one per tile size, inside dev_spans' allocation
  bool coarse_tables = false;                // several runs: all but the finest are filled when knobs ask for them
  int64_t tiles[4] = {0, 0, 0, 0};           // tiles per group for each tile size
  noloco::SpanCell* dev_cells = nullptr;     // over the table of the finest tiles; points into dev_spans' allocation
  int32_t cell_shift = 0;
  noloco::KernelChoice choice{-1, -1, -1, -1, -1, 0};   // -1 = chosen per launch, see resolve()
  // replica-spread pass: per-tensor tiles (unmerged segments), their partial sums
  int32_t num_segments = 0;                  // as given by the caller, empty ones included
  int64_t seg_tiles_total = 0;
  int64_t seg_tiles_limit = 0;               // tiles as the size limit of the static scratch counts them
  int32_t seg_tile_elems = 0;
  Span* dev_seg_spans = nullptr;             // these five point into dev_spans' allocation
  noloco::SpanCell* dev_seg_cells = nullptr; // over the tiles of dev_seg_spans
  int32_t seg_cell_shift = 0;
  noloco::SegmentTiles* dev_seg_tiles = nullptr;
  noloco::PoolJob* dev_jobs = nullptr;
  int32_t* dev_long_segments = nullptr;
  double* dev_partials = nullptr;            // [seg_tiles_total + num_segments + 1]
  int32_t num_jobs = 0;
  int32_t num_long = 0;

  noloco_launch_plan() = default;
  noloco_launch_plan(const noloco_launch_plan&) = delete;
  noloco_launch_plan& operator=(const noloco_launch_plan&) = delete;
  ~noloco_launch_plan() {
    if (dev_spans != nullptr) (void)hipFree(dev_spans);   // the one device allocation of a plan
  }
};

namespace {

// Builds a plan; may throw std::bad_alloc from the host containers (caught by the C entry point).
noloco_status create_plan(const noloco_arena* arena, noloco_launch_plan** out) {
  std::unique_ptr<noloco_launch_plan> plan(new noloco_launch_plan);
  noloco_status st = noloco::merge_segments(arena->segments, arena->num_segments,
                                            arena->worker_stride, &plan->runs);
  if (st != NOLOCO_OK) return st;
  plan->W = arena->W;
  plan->theta_dtype = arena->theta_dtype;
  plan->stride = arena->worker_stride;
  for (const noloco_segment& r : plan->runs) {
    plan->elements += r.numel;
    if (r.numel >= kLongRun) plan->long_elements += r.numel;
  }

  std::vector<Span> all, one;
  std::vector<noloco::SpanCell> cells;
  const bool several_runs = plan->runs.size() > 1;
  const size_t table_bytes = (plan->runs.size() + 1) * sizeof(Span);
  for (int t = 0; t < 4; ++t) {
    plan->tiles[t] = noloco::build_spans(plan->runs, kTileSizes[t], &one);
    if (!several_runs || t == kFineTile) all.insert(all.end(), one.begin(), one.end());
  }
  if (several_runs) noloco::build_cells(one, &cells, &plan->cell_shift);   // `one` is the finest table
  // Table for the replica-spread pass: one span per non-empty segment in the caller's order,
  // cut into tiles of its own, so that every tile lies inside one tensor.
  plan->num_segments = arena->num_segments;
  std::vector<noloco_segment> nonempty;
  std::vector<noloco::SegmentTiles> seg_tiles(static_cast<size_t>(arena->num_segments));
  for (int32_t i = 0; i < arena->num_segments; ++i)
    if (arena->segments[i].numel > 0) nonempty.push_back(arena->segments[i]);
  const int64_t seg_span_offset = static_cast<int64_t>(all.size());
  // The partial sums of 1024-column tiles have to find room in the static scratch where those of the tiles that its
  // limit counts would: else they are taken four at a time, as in large arenas of two rows.
  plan->seg_tile_elems = noloco::spread_tile_elems_for(arena->W);
  plan->seg_tiles_total = plan->seg_tiles_limit = noloco::build_spans(nonempty, plan->seg_tile_elems, &one);
  if (plan->seg_tile_elems > noloco::kSpreadColumns) {
    std::vector<Span> fine;
    const int64_t tiles = noloco::build_spans(nonempty, noloco::kSpreadColumns, &fine);
    const bool fits = tiles + plan->num_segments + 1 <= noloco::kSpreadScratchDoubles;
    const bool pairs = arena->W == 2 && plan->seg_tiles_limit >= kSpreadPairTiles &&
                       8 * plan->elements >= 5 * plan->seg_tiles_limit * plan->seg_tile_elems;
    if (fits && !pairs) {
      plan->seg_tile_elems = noloco::kSpreadColumns;
      plan->seg_tiles_total = tiles;
      one.swap(fine);
    }
  }
  std::vector<noloco::SpanCell> seg_cells;
  if (!nonempty.empty()) noloco::build_cells(one, &seg_cells, &plan->seg_cell_shift, plan->seg_tile_elems);
  all.insert(all.end(), one.begin(), one.end());
  for (int32_t i = 0, k = 0; i < arena->num_segments; ++i) {
    noloco::SegmentTiles& tiles = seg_tiles[static_cast<size_t>(i)];
    tiles.numel = arena->segments[i].numel;
    if (tiles.numel > 0) {
      tiles.first_tile = one[static_cast<size_t>(k)].tile_prefix;
      tiles.num_tiles = one[static_cast<size_t>(k) + 1].tile_prefix - tiles.first_tile;
      ++k;
    } else {
      tiles.first_tile = tiles.num_tiles = 0;
    }
  }
  if (plan->seg_tiles_limit > noloco::kMaxGridWorkgroups) return NOLOCO_ERR_UNSUPPORTED;
  std::vector<noloco::PoolJob> jobs;
  std::vector<int32_t> long_segments;
  noloco::build_pool_jobs(seg_tiles, &jobs, &long_segments);
  plan->num_jobs = static_cast<int32_t>(jobs.size());
  plan->num_long = static_cast<int32_t>(long_segments.size());

  // One device allocation, filled by one copy: span tables, per-segment tile ranges, pooling jobs; then
  // the partial sums, which are written before they are read.
  std::vector<char> tables;
  auto append = [&tables](const void* data, size_t bytes) {
    const size_t at = tables.size();
    tables.resize((at + bytes + 255) / 256 * 256);
    if (bytes > 0) std::memcpy(tables.data() + at, data, bytes);
    return at;
  };
  append(all.data(), all.size() * sizeof(Span));
  const size_t segs_at = append(seg_tiles.data(), seg_tiles.size() * sizeof(noloco::SegmentTiles));
  const size_t jobs_at = append(jobs.data(), jobs.size() * sizeof(noloco::PoolJob));
  const size_t cells_at = append(cells.data(), cells.size() * sizeof(noloco::SpanCell));
  const size_t seg_cells_at = append(seg_cells.data(), seg_cells.size() * sizeof(noloco::SpanCell));
  const size_t long_at = append(long_segments.data(), long_segments.size() * sizeof(int32_t));
  const size_t partial_bytes =
      static_cast<size_t>(plan->seg_tiles_total + plan->num_segments + 1) * sizeof(double);
  const size_t coarse_bytes = several_runs ? (3 * table_bytes + 255) / 256 * 256 : 0;
  char* block = nullptr;
  if (hipGetDevice(&plan->device) != hipSuccess ||
      hipMalloc(reinterpret_cast<void**>(&block), tables.size() + coarse_bytes + partial_bytes) != hipSuccess)
    return NOLOCO_ERR_DEVICE;
  plan->dev_spans = reinterpret_cast<Span*>(block);        // owned from here on (freed by ~noloco_launch_plan)
  plan->dev_seg_spans = plan->dev_spans + seg_span_offset;
  plan->dev_seg_tiles = reinterpret_cast<noloco::SegmentTiles*>(block + segs_at);
  plan->dev_jobs = reinterpret_cast<noloco::PoolJob*>(block + jobs_at);
  plan->dev_cells = reinterpret_cast<noloco::SpanCell*>(block + cells_at);
  plan->dev_seg_cells = reinterpret_cast<noloco::SpanCell*>(block + seg_cells_at);
  plan->dev_long_segments = reinterpret_cast<int32_t*>(block + long_at);
  plan->dev_partials = reinterpret_cast<double*>(block + tables.size() + coarse_bytes);
  for (int t = 0; t < 4; ++t)
    plan->dev_tables[t] = reinterpret_cast<Span*>(several_runs ? (t == kFineTile ? block : block + tables.size() + static_cast<size_t>(t) * table_bytes)
                                                               : block + static_cast<size_t>(t) * table_bytes);
  plan->coarse_tables = !several_runs;
  // A synchronous copy from pageable memory: the tables are final when create returns.
  if (hipMemcpy(block, tables.data(), tables.size(), hipMemcpyHostToDevice) != hipSuccess)
    return NOLOCO_ERR_DEVICE;
  // Resolve this GPU's static scratch array now, at set-up, so that noloco_replica_spread_noalloc
  // finds the address cached.  A failure here only matters to that entry point, which reports it.
  double* unused = nullptr;
  (void)noloco::static_spread_scratch(&unused);
  *out = plan.release();
  return NOLOCO_OK;
}

}  // namespace

extern "C" noloco_status noloco_launch_plan_create(const noloco_arena* arena,
                                                   noloco_launch_plan** out) {
  if (out == nullptr) return NOLOCO_ERR_NULL;
  *out = nullptr;
  if (arena == nullptr) return NOLOCO_ERR_NULL;
  if (arena->phi == nullptr || arena->delta == nullptr || arena->theta == nullptr)
    return NOLOCO_ERR_NULL;
  if (arena->W < 1 || arena->worker_stride < 0 || arena->num_segments < 0)
    return NOLOCO_ERR_INVALID_ARG;
  if (arena->W > NOLOCO_MAX_WORKERS) return NOLOCO_ERR_UNSUPPORTED;
  if (arena->theta_dtype != NOLOCO_F32 && arena->theta_dtype != NOLOCO_BF16)
    return NOLOCO_ERR_INVALID_ARG;
  if (!aligned(arena->phi, NOLOCO_BASE_ALIGN_BYTES) || !aligned(arena->delta, NOLOCO_BASE_ALIGN_BYTES) ||
      !aligned(arena->theta, NOLOCO_BASE_ALIGN_BYTES) ||
      arena->worker_stride % NOLOCO_STRIDE_ALIGN_ELEMS != 0)
    return NOLOCO_ERR_ALIGNMENT;
  try {
    return create_plan(arena, out);
  } catch (const std::bad_alloc&) {
    return NOLOCO_ERR_NO_MEMORY;
  } catch (...) {
    return NOLOCO_ERR_INVALID_ARG;
  }
}

extern "C" noloco_status noloco_launch_plan_destroy(noloco_launch_plan* plan) {
  if (plan == nullptr) return NOLOCO_OK;
  noloco_status st = NOLOCO_OK;
  if (plan->dev_spans != nullptr) {
    if (hipFree(plan->dev_spans) != hipSuccess) st = NOLOCO_ERR_DEVICE;
    plan->dev_spans = nullptr;
  }
  delete plan;
  return st;
}

namespace {

// The tables of the larger tiles of an arena of several runs, which only launches under knobs use.
noloco_status fill_coarse_tables(noloco_launch_plan* plan) {
  try {
    std::vector<Span> all, one;
    for (int t = 0; t < kFineTile; ++t) {
      (void)noloco::build_spans(plan->runs, kTileSizes[t], &one);
      all.insert(all.end(), one.begin(), one.end());
    }
    if (hipMemcpy(plan->dev_tables[0], all.data(), all.size() * sizeof(Span), hipMemcpyHostToDevice) != hipSuccess)
      return NOLOCO_ERR_DEVICE;
  } catch (const std::bad_alloc&) {
    return NOLOCO_ERR_NO_MEMORY;
  } catch (...) {
    return NOLOCO_ERR_INVALID_ARG;
  }
  plan->coarse_tables = true;
  return NOLOCO_OK;
}

}  // namespace

extern "C" noloco_status noloco_launch_plan_tune(noloco_launch_plan* plan,
                                                 const noloco_tuning* tuning) {
  if (plan == nullptr || tuning == nullptr) return NOLOCO_ERR_NULL;
  const int32_t v = tuning->vectors_per_thread;
  if (v != -1 && v != 1 && v != 2 && v != 4) return NOLOCO_ERR_INVALID_ARG;
  if (tuning->nontemporal < -1 || tuning->nontemporal > 1) return NOLOCO_ERR_INVALID_ARG;
  if (tuning->group_major < -1 || tuning->group_major > 1) return NOLOCO_ERR_INVALID_ARG;
  if (tuning->xcd_map < -1 || tuning->xcd_map > 4096) return NOLOCO_ERR_INVALID_ARG;
  const noloco::KernelChoice choice{v, tuning->nontemporal, tuning->group_major, tuning->xcd_map, -1, 0};
  if (resolve(choice, 2, 0).in_order == 0 && !plan->coarse_tables) {
    const noloco_status st = fill_coarse_tables(plan);
    if (st != NOLOCO_OK) return st;
  }
  plan->choice = choice;
  return NOLOCO_OK;
}

namespace {

// Which of the plan's tables a launch uses.  In order, a tile of several runs is one piece: short runs would
// leave most of a larger one empty, and the table of cells stands for pieces.
int tile_table(const noloco_launch_plan* plan, const noloco::KernelChoice& choice, int32_t n) {
  if (choice.in_order != 0 && plan->runs.size() > 1) return kFineTile;
  const int32_t elems = noloco::tile_elems_for(n, choice.vectors_per_thread);
  int t = 0;
  while (kTileSizes[t] != elems) ++t;
  return t;
}

}  // namespace

extern "C" noloco_status noloco_launch_plan_info(const noloco_launch_plan* plan,
                                                 int64_t* elements_per_worker, int32_t* num_runs,
                                                 int64_t* num_tiles, int32_t* tile_elems) {
  if (plan == nullptr) return NOLOCO_ERR_NULL;
  // the work items of a launch of pairs, all workers in one
  const noloco::KernelChoice choice = resolve(plan->choice, 2, plan->tiles[2] * (plan->W / 2));
  const int t = tile_table(plan, choice, 2);
  if (elements_per_worker) *elements_per_worker = plan->elements;
  if (num_runs) *num_runs = static_cast<int32_t>(plan->runs.size());
  if (num_tiles) *num_tiles = plan->tiles[t];
  if (tile_elems) *tile_elems = kTileSizes[t];
  return NOLOCO_OK;
}

namespace {

// Sorted member lists of the groups of one size, gathered into the member table of a launch: one kernel launch, or one per
// tile range if the grid would be too large.
struct LaunchBatch {
  noloco::StepArgs args;
  noloco::KernelChoice choice;
  int32_t theta_dtype;
  void* stream;
  int64_t tiles_total;       // tiles per group for this tile size
  int32_t groups = 0;        // gathered

  noloco_status launch() {
    // A launch holds at most kMaxGridWorkgroups work items: all tiles of `groups` groups if they
    // fit, else a range of tiles at a time.
    const int64_t tiles_per_launch = std::min<int64_t>(tiles_total, noloco::kMaxGridWorkgroups / groups);
    args.num_groups = groups;
    for (int64_t t0 = 0; t0 < tiles_total; t0 += tiles_per_launch) {
      args.tile_offset = t0;
      args.num_tiles = std::min(tiles_per_launch, tiles_total - t0);
      args.work_items = static_cast<uint32_t>(args.num_tiles * groups);
      if (noloco::launch_outer_step(args, theta_dtype, choice, stream) != 0) return NOLOCO_ERR_DEVICE;
    }
    return NOLOCO_OK;
  }
};

}  // namespace

extern "C" noloco_status noloco_outer_step(const noloco_launch_plan* plan, const noloco_arena* arena,
                                           const noloco_hparams* hparams, const int32_t* members,
                                           const int32_t* group_offsets, int32_t num_groups,
                                           void* hip_stream) {
  // No heap allocation and nothing that can throw on this path: all scratch is on the stack.
  if (plan == nullptr || arena == nullptr || hparams == nullptr) return NOLOCO_ERR_NULL;
  if (arena->phi == nullptr || arena->delta == nullptr || arena->theta == nullptr)
    return NOLOCO_ERR_NULL;
  if (num_groups < 0) return NOLOCO_ERR_INVALID_ARG;
  if (num_groups > 0 && (members == nullptr || group_offsets == nullptr)) return NOLOCO_ERR_NULL;
  if (arena->W != plan->W || arena->worker_stride != plan->stride ||
      arena->theta_dtype != plan->theta_dtype)
    return NOLOCO_ERR_INVALID_ARG;
  if (!aligned(arena->phi, NOLOCO_BASE_ALIGN_BYTES) || !aligned(arena->delta, NOLOCO_BASE_ALIGN_BYTES) ||
      !aligned(arena->theta, NOLOCO_BASE_ALIGN_BYTES))
    return NOLOCO_ERR_ALIGNMENT;
  {
    // The step is in place and every array is both read and written: the three must be disjoint.
    const uint64_t elems = static_cast<uint64_t>(plan->W) * static_cast<uint64_t>(plan->stride);
    const uint64_t f32_bytes = elems * 4, theta_bytes = elems * (plan->theta_dtype == NOLOCO_BF16 ? 2 : 4);
    if (overlap(arena->phi, f32_bytes, arena->delta, f32_bytes) ||
        overlap(arena->phi, f32_bytes, arena->theta, theta_bytes) ||
        overlap(arena->delta, f32_bytes, arena->theta, theta_bytes))
      return NOLOCO_ERR_INVALID_ARG;
  }

  // Validate the grouping completely before anything is launched.  `seen` is a bitmap over the
  // workers (plan creation bounds W by NOLOCO_MAX_WORKERS); `count_of_size[n]` counts groups of size n.
  if (num_groups > 0 && group_offsets[0] != 0) return NOLOCO_ERR_BAD_GROUPING;
  uint64_t seen[NOLOCO_MAX_WORKERS / 64];
  std::memset(seen, 0, (static_cast<size_t>(plan->W) + 63) / 64 * sizeof(uint64_t));
  int32_t count_of_size[NOLOCO_MAX_GROUP + 1];
  std::memset(count_of_size, 0, sizeof(count_of_size));
  bool too_large = false;
  int32_t sizes = 0, least = NOLOCO_MAX_GROUP, most = 0, rows = 0, groups_in_use = 0;     // distinct sizes, their range, members, groups
  for (int32_t g = 0; g < num_groups; ++g) {
    const int32_t lo = group_offsets[g], hi = group_offsets[g + 1];
    if (hi < lo) return NOLOCO_ERR_BAD_GROUPING;
    for (int32_t a = lo; a < hi; ++a) {
      const int32_t w = members[a];
      if (w < 0 || w >= plan->W) return NOLOCO_ERR_BAD_GROUPING;
      const uint64_t bit = 1ull << (w & 63);
      if (seen[w >> 6] & bit) return NOLOCO_ERR_BAD_GROUPING;
      seen[w >> 6] |= bit;
    }
    const int32_t n = hi - lo;
    if (n > NOLOCO_MAX_GROUP) too_large = true;
    else if (n > 0) {
      sizes += count_of_size[n]++ == 0 ? 1 : 0;
      least = std::min(least, n);
      most = std::max(most, n);
      rows += n;
      ++groups_in_use;
    }
  }
  if (too_large) return NOLOCO_ERR_UNSUPPORTED;
  if (plan->elements == 0 || sizes == 0) return NOLOCO_OK;

  int device = -1;
  if (hipGetDevice(&device) != hipSuccess) return NOLOCO_ERR_DEVICE;
  if (device != plan->device) return NOLOCO_ERR_INVALID_ARG;

  LaunchBatch batch;
  std::memset(&batch.args, 0, sizeof(batch.args));
  batch.theta_dtype = plan->theta_dtype;
  batch.stream = hip_stream;
  noloco::StepArgs& args = batch.args;
  args.phi = arena->phi;
  args.delta = arena->delta;
  args.theta = arena->theta;
  args.stride = plan->stride;
  args.num_spans = static_cast<int32_t>(plan->runs.size());
  args.cell_shift = plan->cell_shift;
  args.run_begin = plan->runs[0].offset;
  args.run_end = args.run_begin + plan->runs[0].numel;
  args.alpha = hparams->alpha;
  args.beta = hparams->beta;
  args.gamma = hparams->gamma;

  const int32_t state = 8 + (plan->theta_dtype == NOLOCO_BF16 ? 2 : 4);       // bytes of a worker's parameter
  const uint64_t between = std::min({distance(arena->phi, arena->delta), distance(arena->phi, arena->theta), distance(arena->delta, arena->theta)});
  const int64_t run = plan->elements / static_cast<int64_t>(plan->runs.size());          // columns of the mean run
  if (plan->choice.nontemporal == 1) args.stores = noloco::kStreaming;                   // as asked for
  else if (plan->elements * plan->W * state <= kKeptBytes) args.stores = run >= kKeptRun ? noloco::kKept : noloco::kStreaming;
  else args.stores = 3 * plan->long_elements > 2 * plan->elements ? noloco::kThrough : noloco::kStreaming;

  noloco::Together together = {};
  const bool share = sizes > 1 && most <= 16 && rows <= noloco::kMixedRows && plan->elements * rows * state <= mixed_bytes(least, most) &&
                     resolve(plan->choice, 2, 0).in_order != 0 && plan->tiles[kFineTile] * groups_in_use <= noloco::kMaxGridWorkgroups;

  // One pass over the groups per distinct size, sizes ascending; a launch takes as many groups
  // as its member table (NOLOCO_MAX_GROUP rows) holds.
  for (int32_t n = 1; n <= NOLOCO_MAX_GROUP; ++n) {
    if (count_of_size[n] == 0) continue;
    const int64_t bytes = plan->elements * count_of_size[n] * n * state;
    const bool apart = bytes >= kApartBytes, near = between < kFarBytes && !apart;
    batch.choice = resolve(plan->choice, n, plan->tiles[2] * count_of_size[n]);
    args.xcd_run = near && n <= 16 ? 1 : n >= 4 && apart ? kApartRun : 0;
    batch.choice.together = share ? &together : nullptr;
    batch.choice.last = n == most;
    args.group_major = batch.choice.group_major;
    args.xcd_map = batch.choice.xcd_map;
    const int t = tile_table(plan, batch.choice, n);
    args.cells = batch.choice.in_order != 0 && plan->runs.size() > 1 ? plan->dev_cells : nullptr;
    args.piece_shift = 0;
    while ((noloco::kPieceElems << args.piece_shift) < kTileSizes[t]) ++args.piece_shift;
    args.first_piece = plan->runs[0].offset / kTileSizes[t] << args.piece_shift;
    args.spans = plan->dev_tables[t];
    batch.tiles_total = plan->tiles[t];
    args.n = n;
    args.inv_n = 1.0f / static_cast<float>(n);
    int32_t g = 0;
    for (int32_t left = count_of_size[n]; left > 0; left -= batch.groups) {
      batch.groups = std::min(left, NOLOCO_MAX_GROUP / n);
      // A launch is paced by its own groups: the last one of a size may have fewer than the others, and alone be too short.
      if (batch.choice.in_order != 0) {
        const bool bf16 = plan->theta_dtype == NOLOCO_BF16;
        const int64_t groups = share ? groups_in_use : batch.groups;
        const int32_t waves = noloco::waves_per_cu(n, bf16, plan->tiles[kFineTile] * groups, plan->elements * groups, apart && n >= 4, near);
        batch.choice.lds = waves != 0 ? noloco::lds_for_waves(waves) : 0;
        args.phases = noloco::Phases{};
        if (args.stores == noloco::kThrough && !share && !(apart && n > 8))
          args.phases = noloco::phases_of_launch(n, bf16, {plan->tiles[kFineTile], plan->elements, static_cast<int64_t>(plan->runs.size()), groups, plan->stride},
                                                between < kThirdsBytes && !apart);
      }
      for (int32_t gathered = 0; gathered < batch.groups && g < num_groups; ++g) {
        const int32_t lo = group_offsets[g];
        if (group_offsets[g + 1] - lo != n) continue;
        int32_t* rows = args.rows + static_cast<size_t>(gathered) * n;
        std::memcpy(rows, members + lo, static_cast<size_t>(n) * sizeof(int32_t));
        std::sort(rows, rows + n);                       // sums run in ascending worker id
        ++gathered;
      }
      const noloco_status st = batch.launch();
      if (st != NOLOCO_OK) return st;
    }
  }
  return NOLOCO_OK;
}

namespace {

// Common body of the two replica-spread entry points: `partials` is where the per-tile and
// per-segment sums are staged (the plan's own buffer, or the static per-GPU array).
noloco_status spread_into(const noloco_launch_plan* plan, const void* x_device, int32_t x_dtype,
                          double* out_std_device, double* partials, void* hip_stream) {
  noloco::SpreadArgs args;
  args.x = x_device;
  args.stride = plan->stride;
  args.spans = plan->dev_seg_spans;
  args.cells = plan->dev_seg_cells;
  args.cell_shift = plan->seg_cell_shift;
  args.W = plan->W;
  args.inv_W = 1.0f / static_cast<float>(plan->W);
  args.tiles = static_cast<uint32_t>(plan->seg_tiles_total);
  args.partials = partials;
  args.run_shift = plan->choice.xcd_map == 0 ? 0 : 1;       // 1: as many as are best
  args.tile_elems = plan->seg_tile_elems;
  args.num_jobs = plan->num_jobs;
  args.jobs = plan->dev_jobs;
  args.long_segments = plan->dev_long_segments;
  args.num_long = plan->num_long;
  args.ticket = reinterpret_cast<uint32_t*>(partials + plan->seg_tiles_total + plan->num_segments);
  args.elements = static_cast<double>(plan->elements);   // below 2^53: exact
  return noloco::launch_replica_spread(args, x_dtype, plan->dev_seg_tiles, plan->num_segments,
                                       out_std_device, hip_stream) == 0
             ? NOLOCO_OK : NOLOCO_ERR_DEVICE;
}

noloco_status check_spread_args(const noloco_launch_plan* plan, const void* x_device, int32_t x_dtype,
                                const double* out_std_device) {
  if (plan == nullptr || x_device == nullptr || out_std_device == nullptr) return NOLOCO_ERR_NULL;
  if (x_dtype != NOLOCO_F32 && x_dtype != NOLOCO_BF16) return NOLOCO_ERR_INVALID_ARG;
  if (!aligned(x_device, NOLOCO_BASE_ALIGN_BYTES) || !aligned(out_std_device, 8))
    return NOLOCO_ERR_ALIGNMENT;
  int device = -1;
  if (hipGetDevice(&device) != hipSuccess) return NOLOCO_ERR_DEVICE;
  if (device != plan->device) return NOLOCO_ERR_INVALID_ARG;
  return NOLOCO_OK;
}

}  // namespace

extern "C" noloco_status noloco_replica_spread(const noloco_launch_plan* plan, const void* x_device,
                                               int32_t x_dtype, double* out_std_device,
                                               void* hip_stream) {
  const noloco_status st = check_spread_args(plan, x_device, x_dtype, out_std_device);
  if (st != NOLOCO_OK) return st;
  return spread_into(plan, x_device, x_dtype, out_std_device, plan->dev_partials, hip_stream);
}

extern "C" noloco_status noloco_replica_spread_noalloc(const noloco_launch_plan* plan,
                                                       const void* x_device, int32_t x_dtype,
                                                       double* out_std_device, void* hip_stream) {
  const noloco_status st = check_spread_args(plan, x_device, x_dtype, out_std_device);
  if (st != NOLOCO_OK) return st;
  // tile sums, then per-segment sums, then the ticket: same staging as the plan's buffer
  if (plan->seg_tiles_limit + plan->num_segments + 1 > noloco::kSpreadScratchDoubles)
    return NOLOCO_ERR_UNSUPPORTED;
  double* scratch = nullptr;
  if (noloco::static_spread_scratch(&scratch) != 0 || scratch == nullptr) return NOLOCO_ERR_DEVICE;
  // Nothing has to start at zero: every slot that is read is written first by this call's kernels.
  return spread_into(plan, x_device, x_dtype, out_std_device, scratch, hip_stream);
}

extern "C" noloco_status noloco_copy_probe(void* dst_device, const void* src_device, int64_t bytes,
                                           void* hip_stream) {
  if (dst_device == nullptr || src_device == nullptr) return NOLOCO_ERR_NULL;
  if (bytes < 0 || bytes % 16 != 0) return NOLOCO_ERR_INVALID_ARG;
  if (!aligned(dst_device, 16) || !aligned(src_device, 16)) return NOLOCO_ERR_ALIGNMENT;
  if (bytes == 0) return NOLOCO_OK;
  return noloco::launch_stream_probe(0, dst_device, src_device, bytes, 0.f, hip_stream) == 0
             ? NOLOCO_OK : NOLOCO_ERR_DEVICE;
}

extern "C" noloco_status noloco_read_probe(const void* src_device, int64_t bytes, void* sink_device,
                                           void* hip_stream) {
  if (src_device == nullptr || sink_device == nullptr) return NOLOCO_ERR_NULL;
  if (bytes < 0 || bytes % 16 != 0) return NOLOCO_ERR_INVALID_ARG;
  if (!aligned(src_device, 16) || !aligned(sink_device, 4)) return NOLOCO_ERR_ALIGNMENT;
  if (bytes == 0) return NOLOCO_OK;
  return noloco::launch_stream_probe(1, sink_device, src_device, bytes, 0.f, hip_stream) == 0
             ? NOLOCO_OK : NOLOCO_ERR_DEVICE;
}

extern "C" noloco_status noloco_fill_probe(void* dst_device, int64_t bytes, float value,
                                           void* hip_stream) {
  if (dst_device == nullptr) return NOLOCO_ERR_NULL;
  if (bytes < 0 || bytes % 16 != 0) return NOLOCO_ERR_INVALID_ARG;
  if (!aligned(dst_device, 16)) return NOLOCO_ERR_ALIGNMENT;
  if (bytes == 0) return NOLOCO_OK;
  return noloco::launch_stream_probe(2, dst_device, nullptr, bytes, value, hip_stream) == 0
             ? NOLOCO_OK : NOLOCO_ERR_DEVICE;
}

extern "C" const char* noloco_strerror(noloco_status status) {
  switch (status) {
    case NOLOCO_OK: return "ok";
    case NOLOCO_ERR_NULL: return "a required pointer is null";
    case NOLOCO_ERR_INVALID_ARG: return "invalid argument";
    case NOLOCO_ERR_BAD_GROUPING: return "groups are not a valid partition";
    case NOLOCO_ERR_SEGMENT_OVERLAP: return "segments overlap or leave the row";
    case NOLOCO_ERR_ALIGNMENT: return "base pointer or worker stride misaligned";
    case NOLOCO_ERR_DEVICE: return "HIP runtime error";
    case NOLOCO_ERR_UNSUPPORTED: return "documented limit exceeded";
    case NOLOCO_ERR_NO_MEMORY: return "host memory allocation failed";
  }
  return "unknown status";
}
