// What noloco_outer_step launches, without a GPU: the library's host code with stand-ins for the HIP runtime calls it makes
// and for the kernel launchers.  Reads calls from standard input, one a line:
//   bf16 W stride between nruns (offset numel)... ngroups size...
// (`between`: bytes from one array's base to the next one's; 0 = as allocated one after the other; the groups hold the
// workers 0, 1, ... in order) and prints one line for each: its launches as
//   n groups in_order together paced stores phases class_shift;
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "noloco.h"
#include "noloco_internal.h"

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
int launch_outer_step(const StepArgs& a, int32_t, const KernelChoice& c, void*) {
  std::printf("%d %d %d %d %d %u %d %u; ", a.n, a.num_groups, c.in_order, c.together != nullptr, c.lds != 0, a.stores, a.phases.per_tick != 0,
              a.phases.class_shift);
  return 0;
}
int launch_replica_spread(const SpreadArgs&, int32_t, const SegmentTiles*, int32_t, double*, void*) { return 0; }
int launch_stream_probe(int, void*, const void*, int64_t, float, void*) { return 0; }
int static_spread_scratch(double** out) { static double slot[4]; *out = slot; return 0; }
}  // namespace noloco

int main() {
  int bf16 = 0, W = 0;
  long long stride = 0, between = 0, count = 0;
  while (std::scanf("%d %d %lld %lld %lld", &bf16, &W, &stride, &between, &count) == 5) {
    std::vector<noloco_segment> segs(static_cast<size_t>(count));
    for (noloco_segment& s : segs) {
      long long offset = 0, numel = 0;
      if (std::scanf("%lld %lld", &offset, &numel) != 2) return 2;
      s = noloco_segment{offset, numel};
    }
    if (std::scanf("%lld", &count) != 1) return 2;
    std::vector<int32_t> offsets(1, 0), members(static_cast<size_t>(W));
    for (int32_t w = 0; w < W; ++w) members[static_cast<size_t>(w)] = w;
    for (long long g = 0; g < count; ++g) {
      int size = 0;
      if (std::scanf("%d", &size) != 1) return 2;
      offsets.push_back(offsets.back() + size);
    }
    const uint64_t base = 1ull << 40, rows = static_cast<uint64_t>(W) * static_cast<uint64_t>(stride) * 4;
    const uint64_t step = between != 0 ? static_cast<uint64_t>(between) : (rows + (2 << 20) - 1) >> 21 << 21;
    const noloco_arena arena = {reinterpret_cast<float*>(base), reinterpret_cast<float*>(base + step), reinterpret_cast<void*>(base + 2 * step),
                                stride, W, bf16 ? NOLOCO_BF16 : NOLOCO_F32, segs.data(), static_cast<int32_t>(segs.size())};
    const noloco_hparams hp = {0.9f, 0.7f, 1.0f};
    noloco_launch_plan* plan = nullptr;
    if (noloco_launch_plan_create(&arena, &plan) != NOLOCO_OK) return 3;
    const noloco_status status = noloco_outer_step(plan, &arena, &hp, members.data(), offsets.data(), static_cast<int32_t>(count), nullptr);
    if (noloco_launch_plan_destroy(plan) != NOLOCO_OK || status != NOLOCO_OK) return 4;
    std::printf("\n");
  }
  return 0;
}
