// Host check of how workgroups find their columns (built and run by tests/test_pieces.py): over many
// run layouts, the table of cells and the binary search, for every tile size, must each hand out every
// owned column exactly once and no other.
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>

#include "noloco_internal.h"

using namespace noloco;

// A span table that counts how often another of its entries is looked at: what a workgroup would load.
struct CountedSpans {
  const Span* at;
  static const Span* last;
  static int loads;
  static const Span& look(const Span* p) {
    if (p != last) ++loads;
    last = p;
    return *p;
  }
  const Span& operator[](int64_t i) const { return look(at + i); }
  const Span* operator->() const { return &look(at); }
  CountedSpans operator+(int64_t i) const { return CountedSpans{at + i}; }
  CountedSpans& operator++() { ++at; return *this; }
};
const Span* CountedSpans::last = nullptr;
int CountedSpans::loads = 0;

// Arenas with one very long run among many short ones: the cells are sized by the mean run, so one cell
// holds hundreds of runs.  Every tile of a short run must be found as the binary search finds it, with
// no more looks at the table than a binary search over the runs of one cell takes.
static bool skewed(int64_t long_run, int64_t short_run, int64_t count, bool long_first) {
  std::vector<noloco_segment> runs;
  int64_t at = 0;
  for (int64_t i = 0; i <= count; ++i) {
    const int64_t numel = i == (long_first ? 0 : count) ? long_run : short_run;
    runs.push_back(noloco_segment{at, numel});
    at += numel + 300;
  }
  std::vector<Span> spans;
  const int64_t tiles = build_spans(runs, kPieceElems, &spans);
  std::vector<SpanCell> table;
  int32_t cell_shift = 0;
  build_cells(spans, &table, &cell_shift);
  int bound = 2;
  while ((int64_t{1} << (bound - 2)) < count + 1) ++bound;
  const int64_t long_tiles = long_run / kPieceElems, step = std::max<int64_t>(1, long_tiles / 1000);
  for (int64_t t = 0; t < tiles;) {
    Piece a, b;
    CountedSpans::last = nullptr;
    CountedSpans::loads = 0;
    const bool any = locate_by_cells(table.data(), cell_shift, CountedSpans{spans.data()}, t, a);
    if (CountedSpans::loads > bound) { std::printf("tile %lld: %d looks\n", static_cast<long long>(t), CountedSpans::loads); return false; }
    if (any != locate_by_search(spans.data(), static_cast<int32_t>(runs.size()), 0, t, 0, b)) return false;
    if (any && (a.base != b.base || a.lo != b.lo || a.hi != b.hi)) return false;
    const bool inside_long = long_first ? t + step < long_tiles : t >= tiles - long_tiles;
    t += inside_long ? step : 1;
  }
  return true;
}

static bool covers(const std::vector<noloco_segment>& runs, int64_t stride, int32_t tile_elems, bool cells) {
  std::vector<Span> spans;
  const int64_t tiles = build_spans(runs, tile_elems, &spans);
  std::vector<SpanCell> table;
  int32_t cell_shift = 0, piece_shift = 0;
  if (cells) build_cells(spans, &table, &cell_shift);
  while ((kPieceElems << piece_shift) < tile_elems) ++piece_shift;
  std::vector<int> seen(static_cast<size_t>(stride), 0);
  for (int64_t t = 0; t < tiles; ++t)
    for (uint32_t piece = 0; piece < (1u << piece_shift); ++piece) {
      Piece r;
      const bool any = cells ? locate_by_cells(table.data(), cell_shift, spans.data(), t, r)
                             : locate_by_search(spans.data(), static_cast<int32_t>(runs.size()), piece_shift, t, piece, r);
      if (!any) continue;
      if (r.base % kPieceElems != 0 || r.lo < 0 || r.lo >= r.hi || r.hi > kPieceElems) return false;
      for (int64_t c = r.base + r.lo; c < r.base + r.hi; ++c) {
        if (c < 0 || c >= stride) return false;
        ++seen[static_cast<size_t>(c)];
      }
    }
  for (const noloco_segment& run : runs)
    for (int64_t c = run.offset; c < run.offset + run.numel; ++c) --seen[static_cast<size_t>(c)];
  return std::all_of(seen.begin(), seen.end(), [](int n) { return n == 0; });
}

int main() {
  std::mt19937_64 rng(7);
  auto pick = [&](int64_t lo, int64_t hi) { return lo + static_cast<int64_t>(rng() % static_cast<uint64_t>(hi - lo + 1)); };
  for (int trial = 0; trial < 400; ++trial) {
    const int64_t most = trial % 4 == 0 ? 3 : trial % 4 == 1 ? 300 : trial % 4 == 2 ? 3000 : 20000;
    const int64_t gap = trial % 3 == 0 ? 1 : trial % 3 == 1 ? 7 : 5000;
    std::vector<noloco_segment> runs;
    int64_t at = pick(0, 600);
    const int64_t count = pick(1, trial % 5 == 0 ? 1 : 60);
    for (int64_t i = 0; i < count; ++i) {
      noloco_segment run;
      run.offset = at;
      run.numel = trial % 7 == 0 ? kPieceElems * pick(1, 4) : pick(1, most);
      runs.push_back(run);
      at += run.numel + pick(1, gap);
    }
    const int64_t stride = (at + 63) / 64 * 64;
    for (int32_t tile_elems : {1024, 2048, 4096, kPieceElems})
      if (!covers(runs, stride, tile_elems, false)) { std::printf("search: trial %d tile %d\n", trial, tile_elems); return 1; }
    if (!covers(runs, stride, kPieceElems, true)) { std::printf("cells: trial %d\n", trial); return 1; }
  }
  for (bool long_first : {true, false})
    for (int64_t short_run : {int64_t{kPieceElems}, int64_t{3}, int64_t{700}})
      if (!skewed(1ll << 30, short_run, 1500, long_first)) { std::printf("skewed: run %lld\n", static_cast<long long>(short_run)); return 1; }
  // the order of an in-order launch permutes every round of workgroups
  for (uint32_t run : {0u, 1u, 3u, 64u}) {
    const uint32_t round = in_order_round(run), blocks = 3 * round;
    std::vector<int> seen(blocks, 0);
    for (uint32_t b = 0; b < blocks; ++b) {
      const uint32_t p = piece_of_block(b, run, in_order_swap(run));
      if (p >= blocks || p / round != b / round || seen[p]++) { std::printf("order: run %u block %u\n", run, b); return 1; }
    }
  }
  // tiles of the replica-spread pass: tensors in any order, not merged, found by the cells as the span table says; and
  // the order permutes every round of workgroups
  for (int trial = 0; trial < 200; ++trial)
    for (int32_t tile_elems : {kSpreadColumns, 4 * kSpreadColumns}) {
      std::vector<noloco_segment> tensors;
      int64_t at = pick(0, 3000);
      for (int64_t i = 0, count = pick(1, 50); i < count; ++i) {
        tensors.push_back(noloco_segment{at, pick(1, trial % 3 == 0 ? 10 : trial % 3 == 1 ? 5000 : 60000)});
        at += tensors.back().numel + pick(0, 2);
      }
      std::shuffle(tensors.begin(), tensors.end(), rng);
      std::vector<Span> spans;
      const int64_t tiles = build_spans(tensors, tile_elems, &spans);
      std::vector<SpanCell> table;
      int32_t cell_shift = 0;
      build_cells(spans, &table, &cell_shift, tile_elems);
      size_t span = 0;
      for (int64_t t = 0; t < tiles; ++t) {
        while (spans[span + 1].tile_prefix <= t) ++span;
        Piece a, b;
        b.base = (spans[span].first_block + t - spans[span].tile_prefix) * tile_elems;
        if (!cut_to_run(spans[span].col_begin, spans[span].col_end, b, tile_elems) ||
            !locate_by_cells(table.data(), cell_shift, spans.data(), t, a, tile_elems) || a.base != b.base || a.lo != b.lo || a.hi != b.hi) {
          std::printf("tiles: trial %d tile %lld\n", trial, static_cast<long long>(t));
          return 1;
        }
      }
    }
  for (uint32_t shift : {0u, 2u, 4u, 8u}) {
    const uint32_t round = kXcds << shift;
    std::vector<int> seen(3 * round, 0);
    for (uint32_t b = 0; b < 3 * round; ++b) {
      const uint32_t t = tile_of_block(b, shift);
      if (t >= 3 * round || t / round != b / round || seen[t]++) { std::printf("tile order: shift %u block %u\n", shift, b); return 1; }
    }
  }
  // replica spread: float rows are paced from so many rounds of the chip on, where the tensors fill three quarters of the
  // tiles; bf16 rows and tiles of four steps never
  {
    const int32_t want[17] = {0, 0, 0, 7, 5, 4, 4, 3, 3, 3, 3, 3, 3, 3, 3, 3, 3};
    const int64_t many = 1 << 24;
    for (int32_t W = 1; W <= 100; ++W)
      for (int32_t elems : {kSpreadColumns, 4 * kSpreadColumns}) {
        const int32_t k = W <= 16 && elems == kSpreadColumns ? want[W] : 0;
        const int64_t enough = (W >= 10 ? 5 : 10) * kCus * k;
        if (spread_workgroups_per_cu(W, true, many, many * elems, elems) != 0 || spread_workgroups_per_cu(W, false, many, many * elems, elems) != k ||
            spread_workgroups_per_cu(W, false, many, many * elems / 4 * 3, elems) != k ||
            spread_workgroups_per_cu(W, false, many, many * elems / 4 * 3 - 1, elems) != 0 ||
            (k != 0 && (spread_workgroups_per_cu(W, false, enough, enough * elems, elems) != k ||
                        spread_workgroups_per_cu(W, false, enough - 1, (enough - 1) * elems, elems) != 0))) {
          std::printf("spread: W = %d\n", W);
          return 1;
        }
      }
  }
  // a paced launch's claim: so many waves fit a CU's LDS; one more does not (or a larger claim would shut out
  // the last of them), and no smaller claim does that
  for (int32_t waves = 2; waves <= 20; ++waves) {
    const int32_t claim = static_cast<int32_t>(lds_for_waves(waves));
    const bool ok = claim % kLdsUnit == 0 && waves * claim <= kLdsBytes &&
                    ((waves + 1) * claim > kLdsBytes || waves * (claim + kLdsUnit) > kLdsBytes) &&
                    (waves + 1) * (claim - kLdsUnit) <= kLdsBytes;
    if (!ok) { std::printf("lds: %d waves claim %d each\n", waves, claim); return 1; }
  }
  // which launches are paced: by how often their waves fill the chip, not by bytes, and with more waves where
  // runs are much shorter than a piece
  {
    const int64_t cus = kCus;
    bool ok = true;
    auto expect = [&ok](int32_t got, int32_t want, const char* what) {
      if (got != want) { std::printf("waves: %s: %d, not %d\n", what, got, want); ok = false; }
    };
    auto whole = [](int32_t n, bool bf16, int64_t pieces) { return waves_per_cu(n, bf16, pieces, pieces * kPieceElems, false); };
    for (int32_t n : {1, 2, 3, 4, 5, 6, 7, 8, 12, 16, 17, 24, 64, 65, 128, 256})
      for (bool bf16 : {false, true}) {
        const int32_t waves = whole(n, bf16, 1 << 24);
        if (waves < (bf16 ? 3 : 2) || waves > 24) { std::printf("waves: n = %d: %d\n", n, waves); return 1; }
        const int64_t enough = (cus * waves * (n <= (bf16 ? 4 : 6) ? 14 : n > 16 ? 7 : !bf16 ? 24 : n < 8 ? 22 : 26) + 3) / 4;
        expect(whole(n, bf16, enough), waves, "long enough");
        expect(waves_per_cu(n, bf16, 1 << 24, (1ll << 24) * kPieceElems, true), std::max(waves, 4), "apart");
        expect(whole(n, bf16, enough - 1), 0, "too short");
        expect(waves_per_cu(n, bf16, 1 << 24, (3ll << 24) * kPieceElems / 4, false), waves, "three quarters owned");
        const int32_t thin = waves_per_cu(n, bf16, 1 << 24, (1ll << 24) * 65, false);       // 65 of 256 columns
        expect(thin, 4 * waves >= 32 ? 0 : (waves * 256 + 32) / 65, "a quarter owned");
        expect(waves_per_cu(n, bf16, 1 << 24, 1 << 24, false), 0, "one column owned");
      }
    // arrays next to each other: groups of five and more are paced from fewer rounds on, and by n and storage alone
    for (int32_t n = 5; n <= 16; ++n)
      for (bool bf16 : {false, true}) {
        const int32_t waves = bf16 ? (n <= 7 ? 4 : 3) : (n <= 6 ? 3 : 2);
        const int64_t enough = (cus * waves * (n <= 6 ? 14 : bf16 ? 22 : 20) + 3) / 4;
        auto near = [&](int64_t pieces) { return waves_per_cu(n, bf16, pieces, pieces * kPieceElems, false, true); };
        expect(near(1 << 24), waves, "near");
        expect(near(enough), waves, "near, long enough");
        expect(near(enough - 1), 0, "near, too short");
        expect(whole(n, bf16, 1 << 24), bf16 ? (n <= 6 ? 4 : 3) : (n <= 6 ? 3 : 2), "far");
      }
    if (!ok) return 1;
  }
  // launches in phases: which sizes, from how many rounds on; the period is what the launch's bytes take at its rate, and
  // each class has its part of the writing half
  {
    double shortest = 1e9, longest = 0.0, least = 1e9, most = 0.0;
    for (int32_t n = 1; n <= 70; ++n)
      for (bool bf16 : {false, true})
        for (bool near : {false, true})
          for (int64_t runs : {int64_t{1}, int64_t{40}, int64_t{1} << 13}) {
            const LaunchColumns whole = {1 << 20, (int64_t{1} << 20) * kPieceElems, runs, 4, 1 << 28};
            const Phases p = phases_of_launch(n, bf16, whole, near);
            const bool want = n >= (near ? 4 : 2) && n <= (near ? 56 : bf16 ? 24 : 48) && ((n > 4 && near) || runs <= 40);
            const double state = n * (bf16 ? 10.0 : 12.0) * kPieceElems * phase_round(p.class_shift);
            const double rate = 2e-6 * state * p.per_tick / 42949672.96;                      // TB/s
            if ((p.per_tick != 0) != want ||
                (want && (rate < 5.5 || rate > 6.75 || p.class_shift < 2 || p.class_shift > 5 ||
                          p.store_for != (near ? 1u : 2u) * (kHalfPeriod >> p.class_shift)))) {
              std::printf("phases: n = %d: %u, rate %.2f\n", n, p.per_tick, rate);
              return 1;
            }
            if (!want) continue;
            const double per_cu = state / kCus / 1024, period = 42.94967296 / p.per_tick * 1e6;         // KiB, us
            shortest = std::min(shortest, period), longest = std::max(longest, period);
            least = std::min(least, per_cu), most = std::max(most, per_cu);
            LaunchColumns c = {1, kPieceElems, 1, 1, 1 << 28};
            while (phases_of_launch(n, bf16, c, near).per_tick == 0) c.columns = ++c.tiles * kPieceElems;
            const Phases q = phases_of_launch(n, bf16, c, near);
            const uint32_t round = phase_round(q.class_shift);
            shortest = std::min(shortest, 42.94967296 / q.per_tick * 1e6);
            least = std::min(least, state / kCus / 1024 * phase_round(q.class_shift) / phase_round(p.class_shift));
            if (c.tiles % round != 0 || c.tiles < 5 * round || c.tiles > 60 * round) {
              std::printf("phases: n = %d from %lld pieces on\n", n, static_cast<long long>(c.tiles));
              return 1;
            }
          }
    if (shortest < 7.0 || longest > 64.0 || least < 96.0 || most > 680.0) {
      std::printf("phases: periods of %.2f to %.2f us, %.0f to %.0f KiB a CU\n", shortest, longest, least, most);
      return 1;
    }
    for (uint32_t shift : {2u, 3u, 4u, 5u})
      for (uint32_t b = 0; b < 3 * phase_round(shift); ++b)
        if (store_phase(b, shift) != kHalfPeriod + (b / kCus % (1u << shift)) * (kHalfPeriod >> shift)) return 1;
  }
  // pooling jobs: every tile of a long tensor in one chunk, every tensor in one batch
  for (int trial = 0; trial < 50; ++trial) {
    std::vector<SegmentTiles> segs(static_cast<size_t>(pick(0, trial % 2 ? 40 : 3000)));
    int64_t tile = 0;
    for (SegmentTiles& s : segs) {
      s.num_tiles = pick(0, 9) == 0 ? kPoolChunk * pick(1, 3) + pick(-1, 1) : pick(0, 9) == 0 ? kPoolShort + pick(-1, 9) : pick(0, 5);
      s.first_tile = tile;
      tile += s.num_tiles;
      s.numel = s.num_tiles;
    }
    std::vector<PoolJob> jobs;
    std::vector<int32_t> long_segments;
    build_pool_jobs(segs, &jobs, &long_segments);
    // a tensor is finished by a job of its own, by a batch that takes it, or from its chunks
    std::vector<int> tiles(static_cast<size_t>(tile), 0), done(segs.size(), 0);
    for (const PoolJob& j : jobs) {
      if (j.kind == PoolJob::kChunk) {
        if (j.count > kPoolChunk) return 1;
        for (int64_t i = j.first; i < j.first + j.count; ++i) ++tiles[static_cast<size_t>(i)];
      } else if (j.kind == PoolJob::kWhole) {
        ++done[static_cast<size_t>(j.first)];
      } else {
        const int64_t longest = j.kind == PoolJob::kBatch ? kPoolChunk : kPoolShort;
        for (int64_t i = j.first; i < j.first + j.count; ++i)
          if (segs[static_cast<size_t>(i)].num_tiles <= longest) ++done[static_cast<size_t>(i)];
      }
    }
    for (int32_t s : long_segments) ++done[static_cast<size_t>(s)];
    for (size_t s = 0; s < segs.size(); ++s) {
      if (done[s] != 1) return 1;
      for (int64_t t = segs[s].first_tile; t < segs[s].first_tile + segs[s].num_tiles; ++t)
        if (tiles[static_cast<size_t>(t)] != (segs[s].num_tiles > kPoolChunk ? 1 : 0)) return 1;
    }
  }
  std::printf("piece driver: ok\n");
  return 0;
}
