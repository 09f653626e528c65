// Multi-tensor dispatch, host side: segment table -> contiguous runs -> tile spans.
//
// The arena of one worker is a row of `worker_stride` elements in which the tensors occupy
// arbitrary, possibly odd-sized and odd-placed ranges.  Touching ranges are merged into runs so
// that a tight-packed arena of thousands of tensors becomes a single stream; every run is
// then cut at multiples of the tile size (in row coordinates, so interior tiles start on
// 16-byte vector boundaries whatever the run's own start is).
#include <algorithm>
#include <new>

#include "noloco_internal.h"

namespace noloco {

noloco_status merge_segments(const noloco_segment* segments, int32_t num_segments,
                             int64_t worker_stride, std::vector<noloco_segment>* runs) {
  runs->clear();
  if (num_segments < 0 || worker_stride < 0) return NOLOCO_ERR_INVALID_ARG;
  if (num_segments > 0 && segments == nullptr) return NOLOCO_ERR_NULL;

  std::vector<noloco_segment> sorted;
  sorted.reserve(static_cast<size_t>(num_segments));
  for (int32_t s = 0; s < num_segments; ++s) {
    const noloco_segment& seg = segments[s];
    if (seg.offset < 0 || seg.numel < 0) return NOLOCO_ERR_INVALID_ARG;
    if (seg.numel > worker_stride || seg.offset > worker_stride - seg.numel)
      return NOLOCO_ERR_SEGMENT_OVERLAP;  // leaves the row
    if (seg.numel > 0) sorted.push_back(seg);
  }
  std::sort(sorted.begin(), sorted.end(), [](const noloco_segment& a, const noloco_segment& b) {
    return a.offset < b.offset;
  });
  for (const noloco_segment& seg : sorted) {
    if (!runs->empty()) {
      noloco_segment& last = runs->back();
      const int64_t last_end = last.offset + last.numel;
      if (seg.offset < last_end) return NOLOCO_ERR_SEGMENT_OVERLAP;
      if (seg.offset == last_end) {
        last.numel += seg.numel;
        continue;
      }
    }
    runs->push_back(seg);
  }
  return NOLOCO_OK;
}

int64_t build_spans(const std::vector<noloco_segment>& runs, int32_t tile_elems,
                    std::vector<Span>* spans) {
  spans->clear();
  int64_t tiles = 0;
  for (const noloco_segment& run : runs) {
    Span sp;
    sp.col_begin = run.offset;
    sp.col_end = run.offset + run.numel;
    sp.first_block = sp.col_begin / tile_elems;
    sp.tile_prefix = tiles;
    const int64_t last_block = (sp.col_end - 1) / tile_elems;
    tiles += last_block - sp.first_block + 1;
    spans->push_back(sp);
  }
  Span sentinel;
  sentinel.col_begin = sentinel.col_end = sentinel.first_block = 0;
  sentinel.tile_prefix = tiles;
  spans->push_back(sentinel);
  return tiles;
}

void build_cells(const std::vector<Span>& spans, std::vector<SpanCell>* cells, int32_t* shift, int32_t tile_elems) {
  const int64_t tiles = spans.back().tile_prefix, runs = static_cast<int64_t>(spans.size()) - 1;
  *shift = 0;
  while ((tiles >> *shift) > 2 * runs && *shift < 31) ++*shift;
  cells->clear();
  int32_t at = 0;
  auto span_of = [&](int64_t tile) {                 // tiles ascend from call to call
    while (spans[static_cast<size_t>(at) + 1].tile_prefix <= tile) ++at;
    return at;
  };
  const int64_t cell_tiles = int64_t{1} << *shift;
  for (int64_t t = 0; t < tiles; t += cell_tiles) {
    SpanCell c = {};
    c.span = span_of(t);
    c.last_span = span_of(std::min(t + cell_tiles, tiles) - 1);
    for (int i = 0; i < 2; ++i) {
      const int64_t index = std::min<int64_t>(c.span + i, runs - 1);     // without a second span no tile asks for it
      const Span& s = spans[static_cast<size_t>(index)];
      c.block[i] = t + s.first_block - s.tile_prefix;
      c.begin_col[i] = s.tile_prefix >= t ? static_cast<uint32_t>(s.col_begin % tile_elems) : 0u;
      c.end_col[i] = static_cast<uint32_t>((s.col_end - 1) % tile_elems) + 1u;
      c.end_at[i] = static_cast<uint32_t>(std::min<int64_t>(spans[static_cast<size_t>(index) + 1].tile_prefix - t, 0xFFFFFFFFll));
    }
    cells->push_back(c);
  }
}

void build_pool_jobs(const std::vector<SegmentTiles>& segments, std::vector<PoolJob>* jobs,
                     std::vector<int32_t>* long_segments) {
  // Few workgroups, since each draws a ticket, which writes an L2 back: batches in at most 128 (pooling
  // 4096 tensors of 30 000 elements takes 11.2 us with 128, 12.7 with 64, 13.3 with 256), and tensors of
  // more than kPoolShort tiles get one each only while they are few (a wave takes about 1 us for each).
  constexpr int64_t kBatches = 128, kOwnWorkgroups = 96;
  jobs->clear();
  long_segments->clear();
  const int64_t count = static_cast<int64_t>(segments.size());
  int64_t middle = 0;
  for (const SegmentTiles& seg : segments)
    if (seg.num_tiles > kPoolShort && seg.num_tiles <= kPoolChunk) ++middle;
  for (int64_t s = 0; s < count; ++s) {
    const SegmentTiles& seg = segments[static_cast<size_t>(s)];
    if (seg.num_tiles > kPoolChunk) {
      long_segments->push_back(static_cast<int32_t>(s));
      for (int64_t t = 0; t < seg.num_tiles; t += kPoolChunk)
        jobs->push_back(PoolJob{seg.first_tile + t, static_cast<int32_t>(std::min(kPoolChunk, seg.num_tiles - t)),
                                PoolJob::kChunk});
    } else if (seg.num_tiles > kPoolShort && middle <= kOwnWorkgroups) {
      jobs->push_back(PoolJob{s, 1, PoolJob::kWhole});
    }
  }
  const int64_t batch = kPoolSegments * std::max<int64_t>(1, (count + kPoolSegments * kBatches - 1) / (kPoolSegments * kBatches));
  for (int64_t s = 0; s < count; s += batch)
    jobs->push_back(PoolJob{s, static_cast<int32_t>(std::min(batch, count - s)),
                            middle <= kOwnWorkgroups ? PoolJob::kShortBatch : PoolJob::kBatch});
}

// The tile size that the replica-spread pass states its limit of size in.
int32_t spread_tile_elems_for(int32_t W) {
  return (W == 2 || W == 4 || W == 8) ? 4 * kSpreadColumns : kSpreadColumns;
}

// Runs of tiles fill all 16 channels of an XCD's L2, and unlike one contiguous eighth for each XCD they keep the chip in one
// part of the rows.  us, eighths / runs of 4 / 8 / 16 tiles: 60 MB W = 8 float 11.7 / 11.1 / 11.0 / 11.0, W = 24 16.5 / 11.5 / - / 11.5;
// 200 MB W = 16 bf16 36.6 / 31.7 / 30.6 / 30.6; 400 MB W = 32 bf16 67.1 / 60.9 / 59.1 / 58.9, W = 12 float 61.6 / 60.1 / 59.3 / 59.7;
// 4 GB W = 4 float 567 / 586 / 586 / 575; 6.4 GB W = 16 bf16, rows a multiple of 8 KiB apart 894 / 874 / 879 / 890, not so (in
// another allocation) 914 / 901 / - / 891.  Five to seven bf16 rows have no order that they want (4 GB 562 to 568 whichever).
// Few tiles take shorter runs, or some XCDs would have twice as many as others (W = 64 float 60 MB 44.8 / 12.6 / - / 13.5).
// Few rows want longer ones: 4 GB, runs of 16 / 256 tiles W = 1 float 622 / 574, W = 2 598 / 571, bf16 594 / 563, W = 4 bf16 571 / 561
// (200 MB the same, 20 MB 10.6 / 11.4); but not of tiles of 4096 columns (W = 2 bf16 4 GB 549 / 606).
uint32_t spread_run_shift(int32_t W, bool bf16, int64_t tiles, int32_t tile_elems) {
  if (tiles < 1024) return 2;
  if (W <= (bf16 ? 4 : 3) && tiles >= 65536 && tile_elems == kSpreadColumns) return 8;
  return 4;
}

// Reading has a best number of bytes in flight too: about 84 KiB a CU up to seven rows, three workgroups (96 KiB and more)
// above.  us by workgroups per CU (all: as many as fit), 4 GB in one tensor (2 GB in 4096 tensors):
//   W = 3 float all: 573 (301)  8: 554 (291)  7: 546 (286)  6: 550 (295)    W = 4  all: 578 (310)  6: 565 (300)  5: 548 (288)  4: 553 (304)
//   W = 5 float all: 589 (300)  5: 571 (291)  4: 555 (284)  3: 606 (326)    W = 6  all: 590 (298)  5: 580 (293)  4: 566 (288)  3: 583 (307)
//   W = 7 float all: 589 (296)  4: 580 (289)  3: 552 (293)                  W = 8  all: 572 (298)  4: 562 (292)  3: 562 (287)
//   W = 10 float all: 578 (298)  4: 572 (296)  3: 558 (288)                 W = 12 all: 581 (296)  4: 583 (301)  3: 569 (296)  2: 586 (319)
//   W = 16 float all: 571 (298)  4: 574 (294)  3: 558 (288)  2: 565 (306)   W = 24 and more: nothing to gain
// bf16 rows carry half as much per workgroup and are not paced: W = 6 all: 561 (292)  7: 562 (300)  6: 604 (320), W = 7 all: 560 (291)
// 7: 584 (305)  6: 640 (328), W = 8 all: 558 (292)  6: 553 (290), and nothing to gain for W = 3 to 5 and 16.
// Short launches are not paced either; all / paced: ten rounds, W = 4 200 MB 36.1 / 35.2, 120 MB 24.6 / 24.4, W = 7 120 MB 24.5 / 25.8,
// W = 8 200 MB 36.7 / 36.7; from ten rows on five, W = 12 193 MB in 1024 tensors 36.7 / 35.2, 200 MB in one 36.1 / 36.4, W = 11 36.2 / 35.7
// (1024 tensors 36.6 / 35.5), W = 16 120 MB 24.6 / 25.0.
// Tiles that the tensors fill less than three quarters of ask for too little to be held back.  all / paced, tensors over 14 binary
// orders, and how much of the tiles they fill: 400 MB W = 8 0.86 67.7 / 67.1  0.75 70.0 / 73.1  0.60 76.0 / 86.6  0.44 86 / 113  0.18 163 / 283,
// W = 4 0.86 69.7 / 67.7  0.75 74.0 / 75.8  0.60 83 / 94, W = 12 0.80 68.4 / 65.5  0.67 71.6 / 68.7  0.50 77.7 / 81.8; 4 GB W = 6 0.91 599 / 575  0.71 653 / 658,
// W = 10 0.86 597 / 572  0.60 662 / 709.
// Nor have tiles of four steps anything to gain: 4 GB in such tiles W = 4 all: 569  5: 567  4: 565  3: 565  2: 569, W = 8 all: 570  3: 571.
int32_t spread_workgroups_per_cu(int32_t W, bool bf16, int64_t tiles, int64_t columns, int32_t tile_elems) {
  const int32_t k = !bf16 && tile_elems == kSpreadColumns && W >= 3 && W <= 16 ? std::max(3, (21 + W / 2) / W) : 0;
  if (tiles < (W >= 10 ? 5 : 10) * kCus * k || 4 * columns < 3 * tiles * tile_elems) return 0;
  return k;
}

int32_t tile_elems_for(int32_t n, int32_t vectors_per_thread) {
  const int32_t max_u = n <= 2 ? 4 : (n == 4 ? 2 : 1);
  return 1024 * (vectors_per_thread < max_u ? vectors_per_thread : max_u);
}

// Waves of a paced launch that a CU holds: about 48 KiB of loads in flight where the three arrays lie far apart (in
// different thirds of the memory), about 36 KiB where they lie next to each other.
//
// The step reads and writes HBM in equal parts, and with every wave slot filled the requests of some
// thousand workgroups over 3n rows leave the memory no locality.  GB/s by waves per CU.  Up to n = 4: 124 M columns x 16
// rows (12 for n = 3); 5 to 16: 1.5 GB next to each other, 100 to 124 M columns x 10 to 16 rows far apart; 12 M columns from
// n = 24 on, 6 M for n = 100 and 128:
//   next to each other, as dealt             far apart, halves swapped (see piece_of_block())
//   n = 1 float   16: 6455  12: 6658   8: 6649     24: 6589  16: 6623  12: 6642   8: 6586
//   n = 1 bf16    20: 6498  14: 6778  10: 6650     20: 6484  16: 6483  12: 6446
//   n = 2 float    8: 6386   6: 6564   5: 6612     10: 6536   8: 6581   6: 6566   4: 6521
//   n = 2 bf16     8: 6576   7: 6664   5: 6360     10: 6435   8: 6427   6: 6380
//   n = 3 float    5: 6328   4: 6420   3: 6400      7: 6462   5: 6521   4: 6508   3: 6484
//   n = 3 bf16     7: 6356   5: 6526   4: 6265      8: 6426   5: 6400   4: 6221
//   n = 4 float    4: 6250   3: 6365   2: 5884      5: 6492   4: 6521   3: 6514
//   n = 4 bf16     5: 6298   4: 6370   3: 5850      5: 6415   4: 6410   3: 5979
//   n = 5 float    3: 6028   2: 5824                4: 6482   3: 6520
//   n = 5 bf16     5: 5893   4: 5948   3: 5934      4: 6381   3: 6259
//   n = 6 float    3: 5896   2: 5880                4: 6440   3: 6453   2: 6295
//   n = 6 bf16     4: 5851   3: 5804   2: 5236      4: 6496   3: 6427   2: 5496
//   n = 7 float    3: 5687   2: 5857                4: 6398   3: 6415   2: 6473
//   n = 7 bf16     4: 5703   3: 5837                4: 6390   3: 6472   2: 5669
//   n = 8 float    3: 5701   2: 5937                4: 6336   3: 6345   2: 6383
//   n = 8 bf16     3: 5586   2: 5487                4: 6255   3: 6320   2: 5852
//   n = 12 float   3: 5546   2: 5655                4: 6357   3: 6366   2: 6360
//   n = 12 bf16    3: 5364   2: 5372                4: 6368   3: 6357   2: 6022
//   n = 16 float   3: 5342   2: 5427                4: 6289   3: 6278   2: 6274
//   n = 16 bf16    3: 5276   2: 5269                4: 6155   3: 6173   2: 6065
//   n = 24 float  32: 5198    8: 5239   4: 5391   3: 5444      32: 6256   8: 6246   4: 6226   3: 6090
//   n = 24 bf16   32: 5232    8: 5271   5: 5393   4: 5319      32: 6343   8: 6343   5: 6235   4: 6020
//   n = 32 float  32: 5134    8: 5115   4: 5274   3: 5248      32: 6196   8: 6195   4: 6154   3: 5943
//   n = 64 float  32: 5219    8: 5245   4: 5219   3: 5142      32: 6173   8: 6160   4: 6176   3: 5972
//   n = 100 bf16  32: 4853    8: 5068   6: 5106   5: 5112      32: 5843   8: 5906   6: 5895   5: 5787
//   n = 128 float 32: 4813    8: 5037   6: 5074   5: 5115      32: 5700   8: 5918   6: 5983   5: 5926
// bf16 fast weights carry less per wave.  Seven of them next to each other take four waves for the smaller arenas' sake
// (250 MB 92.4 us, three waves 95.4).  Groups of 17 to 64 load eight members at a time (16 KiB), larger ones four; from
// n = 49 on their registers allow four waves anyway.  Arenas of several runs want the same counts (250 MB in runs of 5000,
// us: n = 8 float 3 waves 94.4, 2 89.3; n = 6 float 3 93.8, 2 92.5), but for short ones (see below).
static int32_t paced_waves(int32_t n, bool bf16, bool near) {
  if (n > 64) return 6;
  if (n > 16) return bf16 ? 5 : 4;
  const int32_t least = bf16 ? (n <= (near ? 7 : 6) ? 4 : 3) : n <= 6 ? 3 : 2;
  return std::max(least, ((near ? (bf16 ? 14 : 12) : 16) + n / 2) / n);
}

int32_t waves_per_cu(int32_t n, bool bf16, int64_t pieces, int64_t columns, bool apart, bool near) {
  int32_t waves = paced_waves(n, bf16, near);
  // Arrays in different thirds of the memory want four at least.  ms by waves per CU: 258 GB, bf16, n = 8 3: 81.1
  // 4: 80.9  5: 81.3; n = 16 81.2 81.2 81.3; 269 GB, float, n = 4 3: 85.4  4: 84.6  5: 84.8; n = 8 85.3 85.1 85.2.
  if (apart) waves = std::max(waves, 4);
  // Runs much shorter than a piece leave most of each wave's lanes idle: more waves make up for the bytes
  // that they do not ask for.  250 MB, us by waves per CU, W = 64:
  //   runs of  65 elements  n = 2 8: 232 16: 189 all: 192   n = 8 2: 348  4: 218  8: 194  all: 194
  //   runs of 129 elements  n = 2 8: 155 16: 141 all: 143   n = 8 2: 217  4: 152  8: 145  all: 145
  //   runs of 300 elements  n = 2 8: 108 16: 106 all: 109   n = 8 2: 139  4: 109  8: 111  all: 113
  //   runs of 1000          n = 2 8:  94 16:  99 all: 103   n = 8 2:  98  4: 101  8: 104  all: 106
  // so from pieces owned to three quarters on (runs of some 900 elements) the count is the one above.
  const int64_t whole = pieces * kPieceElems;
  if (4 * columns < 3 * whole) waves = static_cast<int32_t>(std::min<int64_t>(32, (waves * whole + columns / 2) / columns));
  if (waves >= 32) return 0;
  // A short launch is not paced: its last pieces leave most CUs idle, for longer the fewer waves share one.
  // Arenas that are in no cache, us, all waves / paced, and how often the paced waves fill the chip:
  //   n = 2 float 32 MB 14.4 / 14.1 (2.5)  48 MB 20.0 / 19.1 (3.8)  80 MB 31.2 / 29.6 (6.4)
  //   n = 4 float 32 MB 14.1 / 14.4 (2.5)  48 MB 19.6 / 19.2 (3.8)  64 MB 25.6 / 24.7 (5.1)
  //   n = 6 float 64 MB 25.6 / 24.9 (4.5)  80 MB 31.8 / 30.1 (5.7)
  //   n = 6 bf16  48 MB 19.9 / 20.7 (4.1)  64 MB 25.2 / 25.0 (5.4)  80 MB 31.5 / 31.0 (6.8)
  //   n = 8 float 64 MB 25.4 / 25.3 (5.1)  80 MB 32.0 / 30.5 (6.4)
  //   n = 10 float 80 MB 31.1 / 32.3 (5.1) 96 MB 38.1 / 36.7 (6.1) 128 MB 48.3 / 46.7 (8.1)
  //   n = 7 bf16  64 MB 26.9 / 27.4 (4.6)  80 MB 33.9 / 32.1 (5.8)
  //   n = 8 bf16  64 MB 25.7 / 26.5 (4.1)  96 MB 39.6 / 41.3 (6.1) 128 MB 48.3 / 46.7 (8.1)
  //   n = 12 bf16 64 MB 23.8 / 26.2 (2.7) 128 MB 48.0 / 48.4 (5.4) 256 MB 99.0 / 96.8 (10.9)
  //   n = 16 bf16 48 MB 19.0 / 22.2 (1.5) 192 MB 74.4 / 78.0 (6.1) 256 MB 95.3 / 94.4 (8.1)
  //   n = 24 float 96 MB 37.1 / 41.6 (1.3) 128 MB 49.1 / 49.1 (1.7)
  //   n = 32 bf16 128 MB 49.3 / 56.9 (1.2) 192 MB 84.5 / 74.3 (1.8) 256 MB 102.0 / 98.3 (2.4)
  // Next to each other (fewer waves, so more rounds; all waves / paced, rounds):
  //   n = 1 float 8 MB 5.17 / 5.13 (0.9)  16 MB 7.97 / 7.82 (1.7)  50 MB 18.7 / 18.1 (5.3)
  //   n = 2 float 16 MB 8.51 / 8.15 (1.7)  50 MB 19.9 / 18.4 (5.3)   bf16 16 MB 7.97 / 8.08 (1.7)  25 MB 10.9 / 10.9 (2.7)
  //   n = 3 float 16 MB 8.01 / 8.67 (1.7)  25 MB 11.3 / 11.3 (2.7)   bf16 25 MB 11.0 / 11.2 (2.5)  50 MB 20.5 / 19.3 (5.1)
  //   n = 4 float 25 MB 10.9 / 11.4 (2.7)  50 MB 19.9 / 19.0 (5.3)   bf16 50 MB 20.7 / 20.6 (4.8)  80 MB 31.5 / 29.5 (7.6)
  //   n = 5 float 35 MB 13.8 / 14.5 (3.0)  50 MB 19.6 / 19.3 (4.2)   bf16 35 MB 14.9 / 15.5 (2.7)  50 MB 20.5 / 20.0 (3.8)
  //   n = 6 float 35 MB 14.1 / 14.1 (2.5)  50 MB 20.2 / 19.4 (3.5)   bf16 50 MB 20.3 / 20.7 (3.2)  65 MB 26.7 / 25.6 (4.1)
  //   n = 7 float 50 MB 20.4 / 20.9 (4.5)  65 MB 25.4 / 24.6 (5.9)   bf16 80 MB 31.2 / 31.3 (4.4)  110 MB 42.0 / 40.0 (6.0)
  //   n = 8 float 50 MB 18.5 / 19.2 (4.0)  65 MB 25.8 / 24.7 (5.2)   bf16 65 MB 25.5 / 26.2 (4.1)  80 MB 31.7 / 30.3 (5.1)
  //   n = 10 float 65 MB 24.8 / 24.9 (4.1)  80 MB 30.5 / 29.5 (5.1)  bf16 80 MB 31.1 / 31.9 (4.1)  110 MB 44.2 / 41.5 (5.6)
  //   n = 12 float 65 MB 24.8 / 26.1 (3.4)  110 MB 40.4 / 38.7 (5.8)  bf16 110 MB 45.1 / 47.1 (4.7)  150 MB 59.6 / 57.8 (6.4)
  //   n = 14 float 80 MB 31.1 / 32.1 (3.6)  110 MB 42.8 / 42.0 (5.0)  bf16 110 MB 42.6 / 44.5 (4.0)  150 MB 58.1 / 56.2 (5.5)
  //   n = 16 float 80 MB 30.2 / 30.8 (3.2)  110 MB 42.9 / 40.2 (4.4)  bf16 150 MB 64.9 / 68.9 (4.8)
  const int64_t quarter_rounds = 4 * pieces / (kCus * waves);
  int64_t least = n <= (bf16 ? 4 : 6) ? 14 : n > 16 ? 7 : !bf16 ? 24 : n < 8 ? 22 : 26;
  if (near && n <= 4) least = bf16 ? (n == 1 ? 6 : n == 2 ? 10 : 18) : n <= 2 ? 6 : 4 * n;
  else if (near && n <= 16) least = n <= 6 ? 14 : bf16 ? 22 : 20;
  return quarter_rounds >= least ? waves : 0;
}

// Where the arrays lie next to each other, groups of four and more gain by phases.  GB/s of launches of 20 GB, paced as
// above / in phases at the rates below (half as many or twice as many classes):
//   n = 4 float 6329 / 6429          bf16 6244 / 6392 (8: 6206)      n = 5 float 6170 / 6322          bf16 6054 / 6339 (8: 6239)
//   n = 6 float 5876 / 6253          bf16 5912 / 6324 (8: 6230)      n = 8 float 6053 / 6389          bf16 5840 / 6388 (16: 6350)
//   n = 10 float 5838 / 6188         bf16 5652 / 6142                n = 12 float 5644 / 6153         bf16 5656 / 6075 (4: 5575)
//   n = 16 float 5562 / 6173         bf16 5462 / 6065 (4: 5643)      n = 24 float 5278 / 6161         bf16 5304 / 6050
//   n = 32 float 5104 / 6054         bf16 5181 / 5770                n = 48 float 5022 / 6074         bf16 5016 / 5774
//   n = 56 float 5079 / 5968         bf16 5071 / 5775
// and on another card over three allocations n = 4 float 6386 to 6461 / 6428 to 6513  n = 8 6070 to 6096 / 6348 to 6410, bf16 5884 / 6350
// n = 16 5640 to 5657 / 6182 to 6229, 5660 / 6061  n = 24 5277 to 5376 / 6064 to 6119  n = 48 5161 to 5224 / 6023 to 6035, 5110 / 5754  n = 56 4762
// to 5069 / 5957 to 5976, 5007 to 5109 / 5691 to 5732.
// With rows that begin off multiples of 1 KiB n = 4 6066 / 6282, 5987 / 6209, n = 8 5713 / 6267, 5515 / 6274, n = 16 5341 / 6125, 5295 / 5958.
// Arrays that are taken for neighbours and lie in two thirds of the memory all the same (closer than 48 GiB, with the boundary
// between them) are paced at 6100 to 6500, and then phases lose: n = 8 float 6400 / 6400, bf16 6400 / 6330  n = 16 6310 / 6250, 6330 / 6085
// n = 24 bf16 6180 / 6050  n = 32 6160 / 5760  n = 48 6120 / 6050, 6140 / 5765.  By allocation 124 M columns x 16 bf16 rows, n = 16, take 6392 to
// 7320 us paced and 6590 to 6680 in phases (nine allocations).
// Groups of up to three gain nothing next to each other (n = 2 6533 / 6573, n = 3 6410 / 6436, at the best rate each).
// Far apart there is less to gain, with stores that may begin in the next class's part too: n = 4 float 6369 / 6527
// bf16 6404 / 6520, n = 8 6315 / 6522, 6295 / 6484, n = 10 6301 / 6529, 6373 / 6569, n = 16 6155 / 6420, 6214 / 6305, n = 24 6193 / 6480,
// 6205 / 6370, n = 48 float 6143 / 6378; larger bf16 groups nothing (n = 32 6202 / 6262 at the best rate).  Pairs and triples want all 32
// waves: n = 2 float 6516 / 6625 (16 6516), bf16 6544 / 6598 (16 6315), n = 3 6517 / 6593 at 6.8.  Arenas above 96 GiB, whose arrays lie far
// apart by themselves, are alike up to eight members: 258 GB, bf16, ms: n = 2 79.4 / 77.8  n = 4 81.4 / 78.5  n = 8 80.7 / 79.1  n = 16 81.2 / 82.0.
//
// The rate is what the period is cut for.  If memory is slower than that the launch gives way to one without phases, some percent
// slower than a paced one; if it is faster the launch waits.  So it is a little below the best: GB/s by rate, rows at
// multiples of 1 KiB (not at multiples):
//   n = 4 bf16   6300: 6199 (6163)  6400: 6275 (6237)  6500: 6342 (6209)  6600: 6392 (6206)  6700: 6489 (5966)
//   n = 8 float  6300: 6223 (6201)  6400: 6301 (6267)  6500: 6389 (6242)  6600: 6434 (6275)  6700: 6445 (5913)
//   n = 16 float 6100: 6060 (6045)  6200: 6154 (6125)  6300: 6173 (6140)  6400: 6231 (6122)  6500: 6173 (6005)
//   n = 16 bf16  6000: 5958 (5924)  6100: 6039 (5958)  6200: 6065 (5958)  6300: 6110 (5858)  6400: 6062 (5730)
//   n = 24 bf16  6000: 5984 (5978)  6100: 6050 (5974)  6200: 6114 (6056)  6300: 6141 (5741)  6400: 5890 (5467)
//   n = 48 float 6000: 5980 (5980)  6100: 6074 (6078)  6200: 6177 (6140)  6300: 5734 (5580)
//   n = 48 bf16  5800: 5774 (5781)  6000: 5965 (5465)  6100: 5710 (5365)
//
// A launch pays for its phases with most of a period, since it begins anywhere in one.  us, paced / in phases (rounds of the classes):
//   n = 4 float 1 GB 316.0 / 325.7 (20)  2 GB 630.4 / 637.6 (40); larger ones gain
//   n = 6 float 400 MB 134.3 / 134.4 (11)  600 MB 199.1 / 195.4 (16)       bf16 1 GB 333.1 / 325.4 (16)
//   n = 8 float, four classes 400 MB 132.2 / 133.1 (16)  600 MB 196.8 / 195.3 (24)  1 GB 325.7 / 321.1; eight 600 MB 196.8  1 GB 324.8
//   n = 8 bf16 400 MB 138.3 / 136.3 (9.5)  600 MB 204.0 / 196.1 (14)
//   n = 12 float, four classes 400 MB 137.3 / 137.3 (11)  600 MB 205.9 / 205.6 (16)  1 GB 354.6 / 333.9; eight 1 GB 338.2
//   n = 12 bf16 400 MB 143.1 / 146.1 (6.4)  600 MB 213.2 / 210.6 (9.5)
//   n = 16 float, four classes 400 MB 144.1 / 142.0 (8)  1 GB 361.7 / 337.2; eight 400 MB 148.5  1 GB 342.6
//   n = 16 bf16 400 MB 151.0 / 149.1 (4.8)  600 MB 219.3 / 219.0 (7.2)  1 GB 366.1 / 342.3
//   n = 24 float, four classes 300 MB 116.4 / 112.8 (4)  2 GB 742.6 / 672.0; eight 600 MB 225.0 (four 212.2)  2 GB 689.8
//   n = 48 float 400 MB 157.4 / 154.1 (2.6)  600 MB 233.7 / 221.9 (4)     bf16 400 MB 160.5 / 172.0 (3.2)  600 MB 234.4 / 225.2 (4.8)
//
// Pieces that are owned in part disturb the phases.  GB/s, rows at multiples of 1 KiB, paced, then by rate 5600 / 5800 / 6000 / 6200 / 6400:
//   n = 8 float, runs of 12 000 5398: 5560 5712 5837 5545 5246   30 000 5796: 5576 5767 5941 6089 6189   200 000 5938: 5583 5779 5963 6136 6267
//   n = 16 bf16, runs of 12 000 5133: 5494 5583 5497 5233 5123   30 000 5303: 5572 5730 5859 5889 5601   200 000 5348: 5587 5782 5932 6023 5781
//   n = 4 float, runs of 30 000 6154: 5587 5777 5949 6122 6221   200 000 6281: 5589 5785 5967 6156 6287
// so groups of four, and all of arrays far apart (n = 8 float, runs of 30 000, 6230, 6119 at 6450), have phases in long runs only.
Phases phases_of_launch(int32_t n, bool bf16, const LaunchColumns& c, bool near) {
  Phases p = {};
  if (n < (near ? 4 : kPhasedLeast) || n > (near ? kPhasedMost : bf16 ? 24 : 48) || ((n <= 4 || !near) && c.runs > 1 && 400 * c.runs > c.tiles)) return p;
  p.class_shift = n > 24 ? 2 : n <= 3 ? 5 : n <= (bf16 ? 7 : 4) ? 4 : 3;
  const int64_t pieces = c.tiles * c.groups;
  // Floats of a shorter launch want half as many classes.
  if (!bf16 && n >= 8 && p.class_shift == 3 && pieces < 20 * static_cast<int64_t>(phase_round(3))) p.class_shift = 2;
  const int64_t least = !near ? (n <= 8 ? 60 : n <= 24 ? 30 : 15) : n <= 4 ? 48 : n <= 8 ? (bf16 ? 12 : 20) : n <= 16 ? (bf16 ? 8 : 10) : n <= 24 ? (bf16 ? 6 : 5) : 5;
  if (pieces < least * static_cast<int64_t>(phase_round(p.class_shift))) return p;
  double rate = n <= 4 ? 6.6 : n <= 8 ? 6.5 : n <= 16 ? (bf16 ? 6.2 : 6.3) : n <= 24 ? (bf16 ? 6.1 : 6.2) : bf16 ? 5.8 : n <= 48 ? 6.1 : 6.0;   // TB/s
  if (!near) rate = n <= 10 ? 6.7 : n <= 24 ? (bf16 ? 6.5 : 6.65) : 6.4;
  else if (c.stride % kPieceElems != 0 && n <= 24) rate -= 0.1;
  if (c.runs > 1) rate -= 0.05 + 24.0 * static_cast<double>(c.runs) / static_cast<double>(c.tiles);
  if (rate < 5.5) return p;
  const double bytes = 2.0 * n * (bf16 ? 10 : 12) * static_cast<double>(c.columns) / static_cast<double>(c.tiles) * phase_round(p.class_shift);
  p.per_tick = static_cast<uint32_t>(4294967296.0 * rate * 1e4 / bytes);       // 10 ns a tick
  p.store_for = (near ? 1u : 2u) * (kHalfPeriod >> p.class_shift);
  return p;
}

int64_t part_of_launch(const StepArgs& args, int64_t first, StepArgs* part) {
  // Threads of one grid (over all groups, whatever the order): below 2^32, with room for the rounding that
  // the XCD maps add.
  const int64_t threads = static_cast<int64_t>(kStepThreads) << args.piece_shift;
  const int64_t most = (0xFFFFFFFFll - 8 * 4096 * threads) / threads / args.num_groups;
  *part = args;
  part->tile_offset = args.tile_offset + first;
  part->first_piece = args.first_piece + (part->tile_offset << args.piece_shift);
  part->num_tiles = std::min(args.num_tiles - first, most);
  part->work_items = static_cast<uint32_t>(part->num_tiles * part->num_groups);
  part->num_pieces = static_cast<uint32_t>(part->num_tiles << part->piece_shift);
  return part->num_tiles;
}

// A paced workgroup (one wave) claims LDS that it does not use, so that a CU holds no more than `waves` of
// them: the least that does that, which leaves the rest of a CU's LDS to kernels on other streams (two waves
// 52 KiB of the 160, four 30, eight 10).
uint32_t lds_for_waves(int32_t waves) {
  const int32_t one_more = kLdsBytes / (waves + 1) / kLdsUnit * kLdsUnit + kLdsUnit;   // waves + 1 of these do not fit
  return static_cast<uint32_t>(std::min(one_more, kLdsBytes / waves / kLdsUnit * kLdsUnit));
}

}  // namespace noloco

extern "C" noloco_status noloco_merge_segments(const noloco_segment* segments, int32_t num_segments,
                                               int64_t worker_stride, noloco_segment* runs_out,
                                               int32_t* num_runs) {
  if (num_runs == nullptr) return NOLOCO_ERR_NULL;
  *num_runs = 0;
  try {
    std::vector<noloco_segment> runs;
    noloco_status st = noloco::merge_segments(segments, num_segments, worker_stride, &runs);
    if (st != NOLOCO_OK) return st;
    *num_runs = static_cast<int32_t>(runs.size());
    if (runs_out != nullptr) std::copy(runs.begin(), runs.end(), runs_out);
    return NOLOCO_OK;
  } catch (const std::bad_alloc&) {      // no exception leaves the C ABI
    return NOLOCO_ERR_NO_MEMORY;
  } catch (...) {
    return NOLOCO_ERR_INVALID_ARG;
  }
}
