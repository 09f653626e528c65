// Host-only exercise of the library's host code and of the oracle under AddressSanitizer and
// UBSan (built and run by tests/test_host_sanitized.py; no GPU, no HIP runtime).  The C ABI's
// argument checking and launch splitting (api.cpp) run against stand-ins for the few HIP runtime
// calls they make and for the kernel launchers of kernels.hip, which record what would be launched.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "noloco.h"
#include "noloco_internal.h"

using noloco::Span;

// ---- stand-ins: device memory is host memory, launches are recorded ----
extern "C" hipError_t hipGetDevice(int* device) { *device = 0; return hipSuccess; }
extern "C" hipError_t hipMalloc(void** ptr, size_t size) {
  *ptr = std::malloc(size ? size : 1);
  return *ptr ? hipSuccess : hipErrorOutOfMemory;
}
extern "C" hipError_t hipFree(void* ptr) { std::free(ptr); return hipSuccess; }
extern "C" hipError_t hipMemcpy(void* dst, const void* src, size_t size, hipMemcpyKind) {
  std::memcpy(dst, src, size);
  return hipSuccess;
}
namespace noloco {
struct Launch { StepArgs args; KernelChoice choice; };
static std::vector<Launch> launches;
static int fail_at_launch = -1;              // index of the launch the stand-in refuses
int launch_outer_step(const StepArgs& args, int32_t, const KernelChoice& choice, void*) {
  if (static_cast<int>(launches.size()) == fail_at_launch) return 1;
  launches.push_back(Launch{args, choice});
  return 0;
}
static SpreadArgs spread_launch;             // the last one
int launch_replica_spread(const SpreadArgs& args, int32_t, const SegmentTiles*, int32_t, double*, void*) {
  spread_launch = args;
  return 0;
}
int launch_stream_probe(int, void*, const void*, int64_t, float, void*) { return 0; }
int static_spread_scratch(double** out) { static double slot[4]; *out = slot; return 0; }
}  // namespace noloco

extern "C" {
int oracle_plan_groups(uint64_t, uint64_t, int32_t, int32_t, int32_t*, int32_t*);
int oracle_plan_routes(uint64_t, uint64_t, uint64_t, int32_t, int32_t, int32_t*, int32_t*);
int oracle_outer_step_f32(float*, float*, void*, int32_t, int64_t, int32_t, const int64_t*, const int64_t*,
                          int32_t, float, float, float, const int32_t*, const int32_t*, int32_t);
int oracle_replica_spread(const void*, int32_t, int64_t, int32_t, const int64_t*, const int64_t*, int32_t,
                          int32_t, double*);
}

#define CHECK(cond) do { if (!(cond)) { std::printf("CHECK failed at line %d: %s\n", __LINE__, #cond); return 1; } } while (0)

// What the workgroups of a recorded in-order launch would do, cut as the real launcher cuts it: every group
// must get every owned column of the row exactly once, and no other.
static bool covers_in_order(const noloco::StepArgs& args, const std::vector<noloco_segment>& owned, int64_t stride) {
  std::vector<uint8_t> want(static_cast<size_t>(stride), 0);
  for (const noloco_segment& s : owned) std::fill_n(want.begin() + s.offset, s.numel, uint8_t{1});
  std::vector<std::vector<uint8_t>> seen(static_cast<size_t>(args.num_groups), std::vector<uint8_t>(want.size(), 0));
  noloco::StepArgs part;
  for (int64_t t = 0; t < args.num_tiles;) {
    t += noloco::part_of_launch(args, t, &part);
    const uint32_t round = noloco::in_order_round(part.xcd_run), blocks = (part.num_pieces + round - 1) / round * round;
    for (int32_t g = 0; g < part.num_groups; ++g)
      for (uint32_t b = 0; b < blocks; ++b) {
        noloco::Piece r;
        if (!noloco::locate_in_order<const noloco::SpanCell*, const Span*>(part, b, static_cast<uint32_t>(g), r)) continue;
        for (int64_t c = r.base + r.lo; c < r.base + r.hi; ++c) {
          if (c < 0 || c >= stride) return false;
          ++seen[r.group][static_cast<size_t>(c)];
        }
      }
  }
  return std::all_of(seen.begin(), seen.end(), [&](const std::vector<uint8_t>& row) { return row == want; });
}

// The same for a launch under knobs: its tiles, piece by piece, found by the binary search.
static bool covers_by_search(const noloco::StepArgs& args, const std::vector<noloco_segment>& owned, int64_t stride) {
  std::vector<uint8_t> want(static_cast<size_t>(stride), 0), seen(want.size(), 0);
  for (const noloco_segment& s : owned) std::fill_n(want.begin() + s.offset, s.numel, uint8_t{1});
  for (int64_t t = 0; t < args.num_tiles; ++t)
    for (uint32_t piece = 0; piece < (1u << args.piece_shift); ++piece) {
      noloco::Piece r;
      if (!noloco::locate_by_search(args.spans, args.num_spans, args.piece_shift, args.tile_offset + t, piece, r)) continue;
      for (int64_t c = r.base + r.lo; c < r.base + r.hi; ++c) {
        if (c < 0 || c >= stride) return false;
        ++seen[static_cast<size_t>(c)];
      }
    }
  return seen == want;
}

int main() {
  // planners, product against oracle, exact-size buffers so that any overrun is caught
  for (int32_t W : {1, 2, 3, 8, 64, 96, 1000}) {
    for (int32_t n = 1; n <= W; ++n) {
      if (W % n != 0 || (W > 100 && n > 8 && n != W)) continue;
      std::vector<int32_t> m1(W), o1(W / n + 1), m2(W), o2(W / n + 1);
      CHECK(noloco_plan_groups(5, 77, W, n, m1.data(), o1.data()) == NOLOCO_OK);
      CHECK(oracle_plan_groups(5, 77, W, n, m2.data(), o2.data()) == 0);
      CHECK(m1 == m2 && o1 == o2);
    }
  }
  CHECK(noloco_plan_groups(0, 0, 8, 3, nullptr, nullptr) == NOLOCO_ERR_NULL);
  {
    std::vector<int32_t> m(8), o(9);
    CHECK(noloco_plan_groups(0, 0, 8, 3, m.data(), o.data()) == NOLOCO_ERR_BAD_GROUPING);
    CHECK(noloco_plan_groups(~0ull, ~0ull, 8, 8, m.data(), o.data()) == NOLOCO_OK);
  }
  for (int32_t stages : {1, 2, 5}) {
    for (int32_t W : {1, 7, 64}) {
      std::vector<int32_t> s1((stages - 1) * W), r1((stages - 1) * W), s2(s1.size()), r2(r1.size());
      CHECK(noloco_plan_routes(9, 3, 4, stages, W, s1.data(), r1.data()) == NOLOCO_OK);
      CHECK(oracle_plan_routes(9, 3, 4, stages, W, s2.data(), r2.data()) == 0);
      CHECK(s1 == s2 && r1 == r2);
    }
  }
  // segment merging
  {
    std::vector<noloco_segment> segs = {{10, 5}, {0, 10}, {20, 3}, {15, 0}, {23, 1}};
    std::vector<noloco_segment> runs(segs.size());
    int32_t count = -1;
    CHECK(noloco_merge_segments(segs.data(), 5, 64, runs.data(), &count) == NOLOCO_OK && count == 2);
    CHECK(runs[0].offset == 0 && runs[0].numel == 15 && runs[1].offset == 20 && runs[1].numel == 4);
    CHECK(noloco_merge_segments(segs.data(), 5, 23, runs.data(), &count) == NOLOCO_ERR_SEGMENT_OVERLAP);
    CHECK(noloco_merge_segments(nullptr, 0, 64, nullptr, &count) == NOLOCO_OK && count == 0);
    noloco_segment huge = {INT64_MAX - 2, 5};
    CHECK(noloco_merge_segments(&huge, 1, INT64_MAX, nullptr, &count) == NOLOCO_ERR_SEGMENT_OVERLAP);
  }
  // latency model
  {
    double out[4];
    CHECK(noloco_sim_tree_vs_pair(1, 64, 0.0, 0.5, 200, out) == NOLOCO_OK && out[0] > out[2]);
    CHECK(noloco_sim_tree_vs_pair(1, 48, 0.0, 0.5, 200, out) == NOLOCO_ERR_INVALID_ARG);
    CHECK(noloco_sim_barrier_penalty(1, 64, 2, 10, 20, 1.0, 0.7, out) == NOLOCO_OK && out[0] >= out[1]);
  }
  // oracle step and spread on exact-size buffers with ragged segments
  {
    const int32_t W = 6;
    const int64_t S = 64;
    std::vector<float> phi(W * S, 0.5f), delta(W * S, 0.25f), theta(W * S, 0.75f);
    std::vector<uint16_t> theta16(W * S, 0x3F80);
    const int64_t off[3] = {0, 7, 63}, len[3] = {5, 33, 1};
    const int32_t members[6] = {5, 0, 3, 1, 4, 2}, offsets[3] = {0, 4, 6};
    CHECK(oracle_outer_step_f32(phi.data(), delta.data(), theta.data(), 0, S, W, off, len, 3, 0.9f, 0.7f, 1.0f,
                                members, offsets, 2) == 0);
    CHECK(oracle_outer_step_f32(phi.data(), delta.data(), theta16.data(), 1, S, W, off, len, 3, 0.9f, 0.7f, 1.0f,
                                members, offsets, 2) == 0);
    double out[4];
    CHECK(oracle_replica_spread(phi.data(), 0, S, W, off, len, 3, 0, out) == 0);
    CHECK(oracle_replica_spread(theta16.data(), 1, S, W, off, len, 3, 1, out) == 0);
  }
  // ---- the C ABI's host path: validation, bucketing by group size, launch splitting ----
  {
    using noloco::launches;
    float* const phi = reinterpret_cast<float*>(1ull << 40);       // never dereferenced on this path
    float* const delta = reinterpret_cast<float*>(2ull << 40);
    void* const theta = reinterpret_cast<void*>(3ull << 40);
    const noloco_hparams hp = {0.9f, 0.7f, 1.0f};
    auto make_plan = [&](int32_t W, int64_t stride, noloco_launch_plan** plan, noloco_arena* arena) {
      static noloco_segment seg;
      seg = noloco_segment{0, stride};
      *arena = noloco_arena{phi, delta, theta, stride, W, NOLOCO_F32, &seg, 1};
      return noloco_launch_plan_create(arena, plan);
    };
    noloco_launch_plan* plan = nullptr;
    noloco_arena arena;
    // (1) mixed group sizes, members unsorted, a worker left out, an empty group
    CHECK(make_plan(9, 1 << 24, &plan, &arena) == NOLOCO_OK);
    {
      const int32_t members[8] = {7, 2, 5, 0, 3, 1, 8, 6}, offsets[5] = {0, 2, 2, 6, 8};
      launches.clear();
      CHECK(noloco_outer_step(plan, &arena, &hp, members, offsets, 4, nullptr) == NOLOCO_OK);
      CHECK(launches.size() == 2);
      const noloco::StepArgs& a = launches[0].args;            // sizes ascending: the pairs first
      CHECK(a.n == 2 && a.num_groups == 2 && a.inv_n == 0.5f && a.tile_offset == 0);
      CHECK(a.rows[0] == 2 && a.rows[1] == 7 && a.rows[2] == 6 && a.rows[3] == 8);
      CHECK(a.num_tiles == (1 << 24) / 4096 && a.work_items == 2u * a.num_tiles);
      CHECK(launches[0].choice.vectors_per_thread == 4 && a.group_major == 1 && a.xcd_map == 0);
      const noloco::StepArgs& b = launches[1].args;
      CHECK(b.n == 4 && b.num_groups == 1 && b.inv_n == 0.25f);
      CHECK(b.rows[0] == 0 && b.rows[1] == 1 && b.rows[2] == 3 && b.rows[3] == 5);
      CHECK(b.num_tiles == (1 << 24) / 2048 && b.group_major == 0 && b.xcd_map == 1);
      // refused groupings launch nothing
      const int32_t dup[4] = {0, 1, 1, 2}, two[3] = {0, 2, 4}, range[4] = {0, 1, 2, 9};
      const int32_t bad_start[3] = {1, 2, 4}, decreasing[3] = {0, 3, 2};
      launches.clear();
      CHECK(noloco_outer_step(plan, &arena, &hp, dup, two, 2, nullptr) == NOLOCO_ERR_BAD_GROUPING);
      CHECK(noloco_outer_step(plan, &arena, &hp, range, two, 2, nullptr) == NOLOCO_ERR_BAD_GROUPING);
      CHECK(noloco_outer_step(plan, &arena, &hp, members, bad_start, 2, nullptr) == NOLOCO_ERR_BAD_GROUPING);
      CHECK(noloco_outer_step(plan, &arena, &hp, members, decreasing, 2, nullptr) == NOLOCO_ERR_BAD_GROUPING);
      CHECK(noloco_outer_step(plan, &arena, &hp, nullptr, two, 2, nullptr) == NOLOCO_ERR_NULL);
      noloco_arena other = arena;
      other.delta = phi + 64;                                  // aligned, but overlaps phi
      CHECK(noloco_outer_step(plan, &other, &hp, members, offsets, 4, nullptr) == NOLOCO_ERR_INVALID_ARG);
      CHECK(launches.empty());
      CHECK(noloco_outer_step(plan, &arena, &hp, nullptr, nullptr, 0, nullptr) == NOLOCO_OK && launches.empty());
      // the runtime refusing the second launch is reported
      noloco::fail_at_launch = 1;
      CHECK(noloco_outer_step(plan, &arena, &hp, members, offsets, 4, nullptr) == NOLOCO_ERR_DEVICE);
      CHECK(launches.size() == 1);
      noloco::fail_at_launch = -1;
    }
    CHECK(noloco_launch_plan_destroy(plan) == NOLOCO_OK);
    // (2) more groups than one member table holds: 300 pairs go out as 128 + 128 + 44; a group of
    //     257 is refused before anything is launched
    CHECK(make_plan(600, 1 << 20, &plan, &arena) == NOLOCO_OK);
    {
      std::vector<int32_t> members(600), offsets(301);
      for (int32_t w = 0; w < 600; ++w) members[w] = 599 - w;
      for (int32_t g = 0; g <= 300; ++g) offsets[g] = 2 * g;
      launches.clear();
      CHECK(noloco_outer_step(plan, &arena, &hp, members.data(), offsets.data(), 300, nullptr) == NOLOCO_OK);
      CHECK(launches.size() == 3 && launches[0].args.num_groups == 128 && launches[1].args.num_groups == 128 &&
            launches[2].args.num_groups == 44);
      CHECK(launches[2].args.rows[0] == 86 && launches[2].args.rows[1] == 87);   // group 256 = workers {87, 86}
      std::vector<int32_t> big_offsets = {0, 2, 259, 261};
      launches.clear();
      CHECK(noloco_outer_step(plan, &arena, &hp, members.data(), big_offsets.data(), 3, nullptr) == NOLOCO_ERR_UNSUPPORTED);
      CHECK(launches.empty());
    }
    CHECK(noloco_launch_plan_destroy(plan) == NOLOCO_OK);
    // (3) more workgroups than one grid holds: the launch is cut over tile ranges that tile the row
    CHECK(make_plan(2, 1ll << 35, &plan, &arena) == NOLOCO_OK);
    {
      const int32_t members[2] = {1, 0}, offsets[3] = {0, 1, 2};
      for (int32_t vpt : {-1, 1}) {
        const noloco_tuning tuning = {vpt, -1, -1, -1};
        CHECK(noloco_launch_plan_tune(plan, &tuning) == NOLOCO_OK);
        launches.clear();
        CHECK(noloco_outer_step(plan, &arena, &hp, members, offsets, 2, nullptr) == NOLOCO_OK);
        const int64_t tiles = (1ll << 35) / (vpt == 1 ? 1024 : 4096);
        CHECK(launches.size() == (vpt == 1 ? 5u : 2u));
        int64_t next = 0;
        for (const noloco::Launch& l : launches) {
          CHECK(l.args.n == 1 && l.args.num_groups == 2 && l.args.tile_offset == next);
          CHECK(l.args.work_items == static_cast<uint64_t>(l.args.num_tiles) * 2);
          CHECK(static_cast<int64_t>(l.args.work_items) <= noloco::kMaxGridWorkgroups);
          next += l.args.num_tiles;
        }
        CHECK(next == tiles);
      }
    }
    CHECK(noloco_launch_plan_destroy(plan) == NOLOCO_OK);
    // (4) a small arena takes small tiles; limits of plan creation
    CHECK(make_plan(4, 1 << 20, &plan, &arena) == NOLOCO_OK);
    {
      const int32_t members[4] = {0, 1, 2, 3}, offsets[3] = {0, 2, 4};
      launches.clear();
      CHECK(noloco_outer_step(plan, &arena, &hp, members, offsets, 2, nullptr) == NOLOCO_OK);
      CHECK(launches.size() == 1 && launches[0].choice.vectors_per_thread == 1 && launches[0].args.num_tiles == 1024);
    }
    CHECK(noloco_launch_plan_destroy(plan) == NOLOCO_OK);
    // (5) the default dispatch: arenas of one run (odd start and end) and of several, each launch replayed on
    //     the host, as dealt and with the runs per XCD of very large arenas
    for (int32_t runs : {1, 2, 7, 300}) {
      std::vector<noloco_segment> segs;
      int64_t at = 5;
      for (int32_t i = 0; i < runs; ++i) {
        const int64_t numel = runs == 1 ? 200001 : i % 50 == 3 ? 9001 : 1 + (i * 37) % 600;
        segs.push_back(noloco_segment{at, numel});
        at += numel + 1 + (i * 13) % 300;
      }
      const int64_t stride = (at + 63) / 64 * 64;
      arena = noloco_arena{phi, delta, theta, stride, 12, NOLOCO_BF16, segs.data(), runs};
      CHECK(noloco_launch_plan_create(&arena, &plan) == NOLOCO_OK);
      const int32_t members[12] = {0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11}, offsets[5] = {0, 2, 4, 9, 12};
      launches.clear();
      CHECK(noloco_outer_step(plan, &arena, &hp, members, offsets, 4, nullptr) == NOLOCO_OK);
      CHECK(launches.size() == 3);                             // two pairs, a triple, a group of five
      for (const noloco::Launch& l : launches) {
        CHECK(l.choice.in_order == 1 && l.choice.lds == 0 && l.choice.nontemporal == 1 && l.args.xcd_run == 0);
        CHECK((l.args.cells != nullptr) == (runs > 1) && (runs == 1 || l.args.piece_shift == 0));
        CHECK(covers_in_order(l.args, segs, stride));
        noloco::StepArgs apart = l.args;
        apart.xcd_run = 64;
        CHECK(covers_in_order(apart, segs, stride));
        noloco::StepArgs rest = l.args;                        // a launch that begins in the middle of the row
        rest.tile_offset = 1;
        rest.num_tiles -= 1;
        std::vector<noloco_segment> owned = segs;
        int64_t skip = (segs[0].offset / noloco::kPieceElems / (1 << l.args.piece_shift) + 1) * (noloco::kPieceElems << l.args.piece_shift);
        for (noloco_segment& s : owned) {                      // without the first run's first tile
          if (&s != &owned[0]) break;
          const int64_t gone = std::min(s.numel, skip - s.offset);
          s.offset += gone;
          s.numel -= gone;
        }
        CHECK(covers_in_order(rest, owned, stride));
      }
      // what the plan says of its work items is what is launched: 256 columns in several runs, and under a
      // knob the size that was asked for, which every kind of arena then gets
      int64_t tiles = 0, pieces = 0;
      int32_t tile_elems = 0;
      for (const noloco_segment& s : segs) pieces += (s.offset + s.numel - 1) / 256 - s.offset / 256 + 1;
      CHECK(noloco_launch_plan_info(plan, nullptr, nullptr, &tiles, &tile_elems) == NOLOCO_OK);
      CHECK(tiles == launches[0].args.num_tiles && tile_elems == noloco::kPieceElems << launches[0].args.piece_shift);
      CHECK(runs == 1 || (tile_elems == 256 && tiles == pieces));
      for (int32_t vpt : {1, 2, 4}) {
        const noloco_tuning knobs = {vpt, -1, -1, -1};
        CHECK(noloco_launch_plan_tune(plan, &knobs) == NOLOCO_OK);
        launches.clear();
        CHECK(noloco_outer_step(plan, &arena, &hp, members, offsets, 4, nullptr) == NOLOCO_OK && launches.size() == 3);
        CHECK(noloco_launch_plan_info(plan, nullptr, nullptr, &tiles, &tile_elems) == NOLOCO_OK);
        CHECK(tile_elems == 1024 * vpt && tiles == launches[0].args.num_tiles);
        for (const noloco::Launch& l : launches) {
          CHECK(l.choice.in_order == 0 && l.args.cells == nullptr);
          CHECK(noloco::kPieceElems << l.args.piece_shift == (l.args.n == 2 ? 1024 * vpt : 1024));
          CHECK(covers_by_search(l.args, segs, stride));
        }
      }
      CHECK(noloco_launch_plan_destroy(plan) == NOLOCO_OK);
    }
    // (6) which launches are paced and which get runs per XCD, on both sides of either line
    {
      const int32_t members[16] = {0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15};
      const int32_t pairs[9] = {0, 2, 4, 6, 8, 10, 12, 14, 16}, fours[5] = {0, 4, 8, 12, 16}, one[2] = {0, 16};
      auto lds_of = [&](int64_t stride, const int32_t* offsets, int32_t groups, uint32_t* xcd_run, const noloco_tuning* knobs) -> int64_t {
        if (make_plan(16, stride, &plan, &arena) != NOLOCO_OK) return -1;
        if (knobs != nullptr && noloco_launch_plan_tune(plan, knobs) != NOLOCO_OK) return -1;
        launches.clear();
        const bool ok = noloco_outer_step(plan, &arena, &hp, members, offsets, groups, nullptr) == NOLOCO_OK && launches.size() == 1;
        (void)noloco_launch_plan_destroy(plan);
        *xcd_run = ok ? launches[0].args.xcd_run : 99;
        return ok && launches[0].choice.in_order == 1 ? static_cast<int64_t>(launches[0].choice.lds) : -1;
      };
      uint32_t run = 0;
      // eight groups of pairs, eight waves a CU: 3.5 rounds of 2048 pieces are 896 pieces a row
      CHECK(lds_of(896 * 256, pairs, 8, &run, nullptr) == noloco::lds_for_waves(8) && run == 0);
      CHECK(lds_of(895 * 256, pairs, 8, &run, nullptr) == 0);
      CHECK(lds_of(896 * 256, fours, 4, &run, nullptr) == noloco::lds_for_waves(4));
      CHECK(lds_of(895 * 256, fours, 4, &run, nullptr) == 0);
      CHECK(lds_of(3072 * 256, one, 1, &run, nullptr) == noloco::lds_for_waves(2));
      CHECK(lds_of(3071 * 256, one, 1, &run, nullptr) == 0);
      const int64_t third = (96ll << 30) / (16 * 12);          // columns of 96 GiB: a multiple of 64
      CHECK(lds_of(third, pairs, 8, &run, nullptr) == noloco::lds_for_waves(8) && run == 0);
      CHECK(lds_of(third, fours, 4, &run, nullptr) == noloco::lds_for_waves(4) && run == 64);
      CHECK(lds_of(third - 64, fours, 4, &run, nullptr) == noloco::lds_for_waves(4) && run == 0);
      CHECK(lds_of(third, one, 1, &run, nullptr) == noloco::lds_for_waves(4) && run == 64);
      CHECK(lds_of(third - 64, one, 1, &run, nullptr) == noloco::lds_for_waves(2) && run == 0);
      const noloco_tuning streaming = {-1, 1, -1, -1}, ordinary = {-1, 0, -1, -1}, small = {1, -1, -1, -1};
      CHECK(lds_of(third, pairs, 8, &run, &streaming) == noloco::lds_for_waves(8));
      CHECK(lds_of(third, pairs, 8, &run, &ordinary) == -1 && lds_of(third, pairs, 8, &run, &small) == -1);
    }
    // (7) more threads than one grid holds, in order: the parts follow each other without a gap
    CHECK(make_plan(2, 1ll << 35, &plan, &arena) == NOLOCO_OK);
    {
      const int32_t members[2] = {1, 0}, offsets[3] = {0, 1, 2};
      launches.clear();
      CHECK(noloco_outer_step(plan, &arena, &hp, members, offsets, 2, nullptr) == NOLOCO_OK);
      int64_t next = 0;
      for (const noloco::Launch& l : launches) {
        CHECK(l.choice.in_order == 1 && l.args.num_groups == 2);
        noloco::StepArgs part;
        for (int64_t t = 0; t < l.args.num_tiles;) {
          t += noloco::part_of_launch(l.args, t, &part);
          CHECK(static_cast<uint64_t>(part.num_pieces) * part.num_groups * noloco::kStepThreads < 0xFFFFFFFFull);
          noloco::Piece first, last, beyond;
          using Cell = const noloco::SpanCell*;
          CHECK((noloco::locate_in_order<Cell, const Span*>(part, 0, 1, first)) && first.base == next && first.group == 1);
          // the last piece's workgroup: piece_of_block() with xcd_run 0 is its own inverse
          const uint32_t end = noloco::piece_of_block(part.num_pieces - 1, 0, noloco::in_order_swap(0));
          CHECK((noloco::locate_in_order<Cell, const Span*>(part, end, 0, last)) && last.lo == 0 && last.hi == 256);
          CHECK(!(noloco::locate_in_order<Cell, const Span*>(part, noloco::piece_of_block(part.num_pieces, 0, noloco::in_order_swap(0)), 0, beyond)));
          CHECK(last.base + 256 - first.base == static_cast<int64_t>(part.num_pieces) * 256);
          next = last.base + 256;
        }
      }
      CHECK(next == 1ll << 35);
    }
    CHECK(noloco_launch_plan_destroy(plan) == NOLOCO_OK);
    // (8) where the arrays lie: next to each other (bases less than 64 GiB apart, any two of them) the pieces go out as
    //     dealt with fewer waves; and results stay in the memory's cache up to 64 MiB of state, whatever the launch takes
    {
      const int32_t members[16] = {0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15};
      const int32_t pairs[9] = {0, 2, 4, 6, 8, 10, 12, 14, 16}, one_pair[2] = {0, 2};
      struct Seen { uint32_t run, stores, lds; };
      auto launch = [&](int64_t stride, uint64_t delta_at, uint64_t theta_at, const int32_t* offsets, int32_t groups, Seen* seen) {
        if (make_plan(16, stride, &plan, &arena) != NOLOCO_OK) return false;
        arena.delta = reinterpret_cast<float*>((1ull << 40) + delta_at);
        arena.theta = reinterpret_cast<void*>((1ull << 40) + theta_at);
        launches.clear();
        const bool ok = noloco_outer_step(plan, &arena, &hp, members, offsets, groups, nullptr) == NOLOCO_OK && launches.size() == 1;
        if (ok) *seen = Seen{launches[0].args.xcd_run, launches[0].args.stores, launches[0].choice.lds};
        static noloco_segment whole;
        whole = noloco_segment{0, stride};
        const bool covered = !ok || stride > (1 << 22) || covers_in_order(launches[0].args, {whole}, stride);
        (void)noloco_launch_plan_destroy(plan);
        return ok && covered;
      };
      const uint64_t far = 64ull << 30;
      Seen s;
      CHECK(launch(1 << 20, far, 2 * far, pairs, 8, &s) && s.run == 0 && s.lds == noloco::lds_for_waves(8));
      CHECK(launch(1 << 20, far, 2 * far - 256, pairs, 8, &s) && s.run == 1 && s.lds == noloco::lds_for_waves(6));
      CHECK(launch(1 << 20, far - 256, 2 * far, pairs, 8, &s) && s.run == 1);
      CHECK(launch(1 << 20, 3 * far, far - 256, pairs, 8, &s) && s.run == 1 && s.stores == noloco::kThrough);
      const int64_t most = (64ll << 20) / (16 * 12) / 64 * 64;
      CHECK(launch(most, far, 2 * far, pairs, 8, &s) && s.stores == noloco::kKept);
      CHECK(launch(most, far, 2 * far, one_pair, 1, &s) && s.stores == noloco::kKept);
      CHECK(launch(most + 64, far, 2 * far, one_pair, 1, &s) && s.stores == noloco::kThrough);
      // short runs: neither.  What is kept goes by the mean run, what is written through by the share of the columns that
      // lie in runs of 8192 and more: more than two thirds of them
      auto stores_of = [&](const std::vector<int64_t>& runs) {
        std::vector<noloco_segment> segs;
        int64_t at = 0;
        for (int64_t run : runs) {
          segs.push_back(noloco_segment{at, run});
          at += run + 64;
        }
        arena = noloco_arena{phi, delta, theta, (at + 63) / 64 * 64, 16, NOLOCO_F32, segs.data(), static_cast<int32_t>(segs.size())};
        if (noloco_launch_plan_create(&arena, &plan) != NOLOCO_OK) return int64_t{-1};
        launches.clear();
        const bool ok = noloco_outer_step(plan, &arena, &hp, members, pairs, 8, nullptr) == NOLOCO_OK && launches.size() == 1;
        (void)noloco_launch_plan_destroy(plan);
        return ok ? static_cast<int64_t>(launches[0].args.stores) : -1;
      };
      for (int64_t run : {3072, 5000, 8191, 8192, 16383, 16384}) {
        CHECK(stores_of(std::vector<int64_t>(2, run)) == (run >= 16384 ? noloco::kKept : noloco::kStreaming));
        CHECK(stores_of(std::vector<int64_t>(static_cast<size_t>((64ll << 20) / (16 * 12) / run + 1), run)) ==
              (run >= 8192 ? noloco::kThrough : noloco::kStreaming));
      }
      std::vector<int64_t> mixed(200, 1000);
      mixed.push_back(400000);                                 // two thirds exactly
      CHECK(stores_of(mixed) == noloco::kStreaming);
      mixed.back() += 1;
      CHECK(stores_of(mixed) == noloco::kThrough);
      // an explicit nontemporal = 1 is obeyed, whatever the automatic choice would store
      for (int64_t stride : {int64_t{1} << 18, int64_t{1} << 20}) {
        CHECK(make_plan(16, stride, &plan, &arena) == NOLOCO_OK);
        for (int32_t asked : {1, -1}) {
          const noloco_tuning knobs = {-1, asked, -1, -1};
          CHECK(noloco_launch_plan_tune(plan, &knobs) == NOLOCO_OK);
          launches.clear();
          CHECK(noloco_outer_step(plan, &arena, &hp, members, pairs, 8, nullptr) == NOLOCO_OK && launches.size() == 1);
          CHECK(launches[0].choice.in_order == 1);
          CHECK(launches[0].args.stores == (asked == 1 ? noloco::kStreaming : stride == 1 << 18 ? noloco::kKept : noloco::kThrough));
        }
        CHECK(noloco_launch_plan_destroy(plan) == NOLOCO_OK);
      }
      // from six waves of 1.5 rounds of the chip on
      CHECK(launch(288 * 256, 1 << 30, 2ll << 30, pairs, 8, &s) && s.lds == noloco::lds_for_waves(6));
      CHECK(launch(287 * 256, 1 << 30, 2ll << 30, pairs, 8, &s) && s.lds == 0);
      // very large: in different thirds by themselves, whatever the bases say
      const int64_t third = (96ll << 30) / (16 * 12);
      CHECK(launch(third, 34ull << 30, 68ull << 30, pairs, 8, &s) && s.run == 0 && s.lds == noloco::lds_for_waves(8));
      CHECK(launch(third - 64, 34ull << 30, 68ull << 30, pairs, 8, &s) && s.run == 1 && s.lds == noloco::lds_for_waves(6));
    }
    // (9) tiles of the replica-spread pass: 4096 columns for pairs of rows in large arenas whose tensors fill five eighths of
    //     them, and for 2, 4 and 8 rows where the sums of smaller tiles would not fit the static scratch; else 1024
    {
      auto tile_elems = [&](int32_t W, const std::vector<noloco_segment>& segs, int64_t stride) {
        arena = noloco_arena{phi, delta, theta, (stride + 63) / 64 * 64, W, NOLOCO_F32, segs.data(), static_cast<int32_t>(segs.size())};
        if (noloco_launch_plan_create(&arena, &plan) != NOLOCO_OK) return -1;
        double out = 0.0;                                      // its address is all that is passed on
        const bool ok = noloco_replica_spread(plan, phi, NOLOCO_F32, &out, nullptr) == NOLOCO_OK;
        (void)noloco_launch_plan_destroy(plan);
        return ok ? noloco::spread_launch.tile_elems : -1;
      };
      auto tensors = [](int64_t count, int64_t numel, int64_t step) {
        std::vector<noloco_segment> segs;
        for (int64_t i = 0; i < count; ++i) segs.push_back(noloco_segment{i * step, numel});
        return segs;
      };
      for (int32_t W : {1, 2, 3, 4, 8, 16}) {
        CHECK(tile_elems(W, tensors(1, 8192ll * 4096, 1), 8192ll * 4096) == (W == 2 ? 4096 : 1024));
        CHECK(tile_elems(W, tensors(1, 8191ll * 4096, 1), 8191ll * 4096) == 1024);
        CHECK(tile_elems(W, tensors(8192, 100, 4096), 8192ll * 4096) == 1024);          // many tiles, nearly empty
        CHECK(tile_elems(W, tensors(8192, 2560, 4096), 8192ll * 4096) == (W == 2 ? 4096 : 1024));
        CHECK(tile_elems(W, tensors(8192, 2559, 4096), 8192ll * 4096) == 1024);
        std::vector<noloco_segment> segs = tensors(3, 5000, 5001);
        segs.resize((1 << 21) - 1 - 6, noloco_segment{0, 0});
        const bool coarse = W == 2 || W == 4 || W == 8;        // 6 tiles of 4096 columns fit, 17 of 1024 do not
        CHECK(tile_elems(W, segs, 15003) == (coarse ? 4096 : 1024));
        segs.resize((1 << 21) - 1 - 17);
        CHECK(tile_elems(W, segs, 15003) == 1024);
      }
    }
    // (10) launches in phases: three bases half a third of the memory from each other lie in more than one third, and have the
    //      rate and the longer parts of arrays far apart; anything closer may lie in one
    {
      const int32_t members[16] = {0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15}, one[2] = {0, 16}, pairs[9] = {0, 2, 4, 6, 8, 10, 12, 14, 16};
      auto phases_at = [&](uint64_t delta_at, uint64_t theta_at, const int32_t* offsets, int32_t groups, noloco::Phases* p) {
        if (make_plan(16, 1 << 26, &plan, &arena) != NOLOCO_OK) return false;
        arena.delta = reinterpret_cast<float*>((1ull << 40) + delta_at);
        arena.theta = reinterpret_cast<void*>((1ull << 40) + theta_at);
        launches.clear();
        const bool ok = noloco_outer_step(plan, &arena, &hp, members, offsets, groups, nullptr) == NOLOCO_OK && launches.size() == 1;
        if (ok) *p = launches[0].args.phases;
        (void)noloco_launch_plan_destroy(plan);
        return ok;
      };
      const uint64_t half = 48ull << 30;
      for (uint64_t less : {0, 256}) {
        noloco::Phases p;
        CHECK(phases_at(half, 2 * half - less, one, 1, &p) && p.per_tick != 0 && p.store_for == (less ? 1u : 2u) * (noloco::kHalfPeriod >> p.class_shift));
        CHECK(phases_at(2 * half, half - less, one, 1, &p) && p.per_tick != 0 && p.store_for == (less ? 1u : 2u) * (noloco::kHalfPeriod >> p.class_shift));
        CHECK(phases_at(half, 2 * half - less, pairs, 8, &p) && (p.per_tick != 0) == (less == 0));
      }
    }
    // (11) the groups that one member table has no room for go out in a launch of their own, which is paced or in phases as
    //      if it were alone
    for (int32_t rest : {1, 8, 15}) {
      const int32_t W = 256 + 16 * rest;
      for (int64_t stride : {int64_t{1} << 14, int64_t{1} << 17, int64_t{1} << 21}) {
        std::vector<int32_t> members(W), offsets(W / 16 + 1);
        for (int32_t w = 0; w < W; ++w) members[w] = w;
        for (size_t g = 0; g < offsets.size(); ++g) offsets[g] = 16 * static_cast<int32_t>(g);
        CHECK(make_plan(W, stride, &plan, &arena) == NOLOCO_OK);
        launches.clear();
        CHECK(noloco_outer_step(plan, &arena, &hp, members.data(), offsets.data(), W / 16, nullptr) == NOLOCO_OK && launches.size() == 2);
        CHECK(noloco_outer_step(plan, &arena, &hp, members.data(), offsets.data(), rest, nullptr) == NOLOCO_OK && launches.size() == 3);
        CHECK(launches[1].args.num_groups == rest && launches[2].args.num_groups == rest);
        CHECK(launches[1].choice.lds == launches[2].choice.lds && launches[1].args.phases.per_tick == launches[2].args.phases.per_tick);
        CHECK((launches[0].args.phases.per_tick != 0) == (stride == 1 << 21) && (stride == 1 << 14) == (launches[0].choice.lds == 0));
        CHECK(noloco_launch_plan_destroy(plan) == NOLOCO_OK);
      }
    }
    CHECK(make_plan(NOLOCO_MAX_WORKERS + 1, 64, &plan, &arena) == NOLOCO_ERR_UNSUPPORTED && plan == nullptr);
    CHECK(make_plan(4, 63, &plan, &arena) == NOLOCO_ERR_ALIGNMENT);
  }
  std::printf("host sanitize driver: ok\n");
  return 0;
}
