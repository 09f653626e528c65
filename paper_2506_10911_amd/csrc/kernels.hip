// Fused NoLoCo outer step for gfx950 (arxiv 2506.10911, section "Outer optimizer step with
// modified Nesterov momentum", Eq. 1-3, plus the restart of the fast weights).
//
// The operation is a pure stream: per worker-parameter it reads phi, delta, theta once and
// writes them once, with about ten flops in between, so HBM bandwidth is the only roofline
// that matters.  The kernels are therefore organised around memory access:
//   * one thread owns one 16-byte vector of four consecutive columns of ONE subgroup and
//     does the whole step for all n members of it, so every byte is moved exactly once and
//     the subgroup reduction never leaves registers;
//   * a workgroup is one wave and covers one piece, 256 columns: its load instruction covers
//     1 KiB of consecutive addresses of one row (buffer_load_dwordx4; 8 bytes per lane for
//     bf16 theta), and all loads of a thread are issued before the first use (groups of up to 16);
//   * whole pieces are written through the L2, or kept in the memory's cache: see Policy;
//   * the pieces are taken in the order of the arena, and few at a time: see waves_per_cu(); in large launches of
//     larger groups the whole chip reads, then writes: see wait_for_phase();
//   * the first and last vector of a run, owned in part, are loaded whole and stored element by
//     element, so a tensor's edges cost no extra round trip.
//
// Arithmetic contract (binary32, one rounding per operation, no contraction; this file is
// compiled with -ffp-contract=off), members a = 0..n-1 in ascending worker id:
//   D_a = phi_a - widen(theta_a);  SD = D_0 (+ D_a ...);  SP = phi_0 (+ phi_a ...)
//   mD = SD * inv_n;  mP = SP * inv_n
//   delta'_a = (alpha*delta_a - beta*mD) - gamma*(phi_a - mP)
//   phi'_a = phi_a + delta'_a;  theta'_a = narrow(phi'_a)
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstring>
#include <type_traits>

#include "noloco_internal.h"

namespace noloco {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned short h4 __attribute__((ext_vector_type(4)));  // four bf16 bit patterns
typedef __bf16 b4 __attribute__((ext_vector_type(4)));
typedef unsigned int u2 __attribute__((ext_vector_type(2)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));

struct Bf16Tag {};  // theta stored as bf16; `float` doubles as the tag for fp32 theta

// bf16 is the upper half of binary32.  Narrowing rounds to nearest, ties to even, by adding
// 0x7FFF plus the lowest kept bit and dropping 16 bits; NaN is kept as a quiet NaN.
__device__ __forceinline__ unsigned int narrow_bits(unsigned int u) {
  const unsigned int r = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
  const unsigned int q = (u >> 16) | 0x0040u;
  return ((u & 0x7FFFFFFFu) > 0x7F800000u) ? q : r;
}

// How a lane's four columns of `theta` are held in memory.
template <typename Tag> struct ThetaMem;
template <> struct ThetaMem<float> {
  typedef float elem; typedef f4 mem;
  static __device__ __forceinline__ f4 widen(f4 m) { return m; }
  static __device__ __forceinline__ f4 narrow(f4 v) { return v; }
  static __device__ __forceinline__ f4 narrow_at_once(f4 v) { return v; }
};
template <> struct ThetaMem<Bf16Tag> {
  typedef unsigned short elem; typedef h4 mem;
  static __device__ __forceinline__ f4 widen(h4 m) {
    u4 w = __builtin_convertvector(m, u4) << 16;
    return __builtin_bit_cast(f4, w);
  }
  static __device__ __forceinline__ h4 narrow(f4 v) {
    u4 u = __builtin_bit_cast(u4, v);
    u4 r;
    r.x = narrow_bits(u.x); r.y = narrow_bits(u.y); r.z = narrow_bits(u.z); r.w = narrow_bits(u.w);
    return __builtin_convertvector(r, h4);
  }
  // The same for all inputs, one instruction for two elements (v_cvt_pk_bf16_f32).  For outer_step_held, which narrows between its
  // stores: in phases computing there keeps the memory waiting (n = 24 6.09 -> 6.21 TB/s, n = 48 5.5 -> 5.9).  The other kernels
  // narrow before their stores, where nothing waits for it.
  static __device__ __forceinline__ h4 narrow_at_once(f4 v) { return __builtin_bit_cast(h4, __builtin_convertvector(v, b4)); }
};

template <bool NT, typename T> __device__ __forceinline__ T ld(const T* p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool NT, typename T> __device__ __forceinline__ void st(T* p, T v) {
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// How the step's accesses go through the caches (the cache-policy bits of a buffer instruction).
//
// kStoreThrough, sc1 and nt: written through the XCD's L2 at once.  With nt alone (the compiler's non-temporal
// store) the lines stay dirty in the L2 until something evicts them, in an order that HBM has no locality in.  GB/s,
// 124 M columns x 16 float rows, nt / sc1 nt, at the best number of waves of each:
//   arrays next to each other  n = 1 6604 / 6768  n = 2 6425 / 6526  n = 4 6247 / 6313  n = 12 5616 / 5735  n = 16 5455 / 5516
//   far apart                       6639 / 6655       6540 / 6562       6455 / 6500        6364 / 6366        6305 / 6288
// and 258 GB, bf16, ms: n = 2 80.3 / 80.1  n = 4 81.2 / 81.0  n = 8 80.9 / 80.8  n = 16 81.1 / 81.0.  Short runs lose (see kLongRun), and so
// do a few launches of one or two rounds of the chip, by up to 3 % (n = 4 float 30 MB 12.4 / 12.5, n = 16 11.4 / 11.8).
// kStoreKept, sc0 and sc1 without nt: through the L2 too, but kept in the 256 MB cache in front of HBM (see kKeptBytes).
// kStreamed, nt: loads (without it n = 2 6366 -> 6011), and the stores of pieces that are owned in part: written through,
// an edge's vectors and its single elements reach the memory one by one (1024 runs of 4 k elements, n = 2, 125 -> 148 us).
enum Policy : int { kCached = 0, kStreamed = 2, kStoreThrough = 18, kStoreKept = 17 };
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, int32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}

// A wave's piece of one row of an array of E: its address is the same for the whole wave (scalar registers) and a
// lane adds its 32-bit offset, so that no access needs an address in vector registers.
template <typename E> struct RowPiece {
  E* at;
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer() const {
    return buffer_of(at, kPieceElems * static_cast<int32_t>(sizeof(E)));
  }
  template <bool NT, typename V> __device__ __forceinline__ V load(uint32_t lane) const {
    constexpr int policy = NT ? kStreamed : kCached;
    const int32_t offset = static_cast<int32_t>(lane * sizeof(E));
    if constexpr (sizeof(V) == 16) return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(buffer(), offset, 0, policy));
    else return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(buffer(), offset, 0, policy));
  }
  template <int policy, typename V> __device__ __forceinline__ void store(uint32_t lane, V v) const {
    const int32_t offset = static_cast<int32_t>(lane * sizeof(E));
    if constexpr (sizeof(V) == 16) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), buffer(), offset, 0, policy);
    else __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), buffer(), offset, 0, policy);
  }
  __device__ __forceinline__ void store_element(uint32_t column, E v) const {
    const int32_t offset = static_cast<int32_t>(column * sizeof(E));
    if constexpr (sizeof(E) == 4) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), buffer(), offset, 0, kCached);
    else __builtin_amdgcn_raw_buffer_store_b16(v, buffer(), offset, 0, kCached);
  }
};

// Enqueue a kernel and return the launch status itself (hipLaunchKernel), so that an error some
// earlier, unrelated call left behind on this thread is neither reported as ours nor cleared.
template <typename T> struct same { typedef T type; };
template <typename... KArgs>
hipError_t enqueue(void (*kernel)(KArgs...), dim3 grid, dim3 block, uint32_t lds, hipStream_t s,
                   typename same<KArgs>::type... args) {
  void* argv[] = {static_cast<void*>(&args)...};
  return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, argv, lds, s);
}

// Tables that no kernel writes, read through the scalar cache (where the index is the same for a wave).
#define scalar_memory __attribute__((address_space(4)))
template <typename T> __device__ __forceinline__ const scalar_memory T* scalar_pointer(const T* p) {
  return (const scalar_memory T*)(p);
}

// Workgroup -> piece under explicit launch-shape knobs.
__device__ __forceinline__ bool locate_mapped(const StepArgs& a, Piece& r) {
  // The hardware deals consecutive workgroups to the 8 XCDs in turn; the map gives each XCD runs of
  // consecutive pieces instead.
  uint32_t unit = blockIdx.x;
  const uint32_t units = a.work_items << a.piece_shift;
  if (a.xcd_map != 0) {
    const uint32_t xcd = unit % kXcds, slot = unit / kXcds;
    if (a.xcd_map == 1) {
      const uint32_t per_xcd = (units + kXcds - 1) / kXcds;
      unit = xcd * per_xcd + slot;                            // one contiguous range per XCD
    } else {
      const uint32_t c = static_cast<uint32_t>(a.xcd_map) << a.piece_shift;    // runs of c tiles per XCD
      const uint32_t blk = slot / c;
      unit = (blk * kXcds + xcd) * c + (slot - blk * c);
    }
    if (unit >= units) return false;
  }
  const uint32_t item = unit >> a.piece_shift;
  const uint32_t piece = unit - (item << a.piece_shift);
  const uint32_t tiles = static_cast<uint32_t>(a.num_tiles);   // host keeps tiles*groups below the grid limit
  uint32_t local;
  if (a.group_major) {
    r.group = item / tiles;
    local = item - r.group * tiles;
  } else {
    const uint32_t groups = static_cast<uint32_t>(a.num_groups);
    local = item / groups;
    r.group = item - local * groups;
  }
  return locate_by_search(scalar_pointer(a.spans), a.num_spans, a.piece_shift,
                          a.tile_offset + static_cast<int64_t>(local), piece, r);
}

// Arguments of an in-order launch whose groups have ROWS members in all at most.  The shorter they are the less a launch
// costs, and a group or a few of them are what a small arena has: 232 bytes instead of 1.2 KB and everything that a
// workgroup needs to find its columns in one line each of arguments and table took a step of 50 MB from 16.05 to 15.61 us,
// two launches on 566 MB from 155.9 to 154.3 and pairs of 1024 runs from 124.7 to 123.7.
template <int ROWS> struct InOrderArgs {
  float* phi;
  float* delta;
  void* theta;
  int64_t stride;
  InOrderHead head;
  float alpha, beta, gamma, inv_n;
  int32_t n;
  uint32_t stores;
  int32_t rows[ROWS];
};
constexpr int kFewRows = 32;
struct PhasedArgs : InOrderArgs<NOLOCO_MAX_GROUP> {
  Phases phases;
};
struct MixedArgs : InOrderArgs<kMixedRows> {
  uint32_t groups[kMixedRows];           // where a group's rows begin, and its size in the upper half
};
template <typename Args> constexpr bool kPhased = std::is_same<Args, PhasedArgs>::value;
template <typename Args> constexpr bool kInOrder = !std::is_same<Args, StepArgs>::value;

// In the order of the arena, group by group, blockIdx.x counts the pieces and blockIdx.y the groups.  In a paced
// launch few waves share a CU, so their start-up is not hidden by others: it takes no division and one or
// two round trips of scalar loads.  (The general way above takes six and two divisions; pairs of float rows
// then needed twice the waves and ran 4 % behind.)
template <typename Args> __device__ __forceinline__ bool locate(const Args& a, Piece& r) {
  if constexpr (kInOrder<Args>) {
    r.group = blockIdx.y;
    return locate_by_head<const scalar_memory SpanCell*, const scalar_memory Span*>(a.head, blockIdx.x, r);
  } else {
    return locate_mapped(a, r);
  }
}

// A launch in phases.  HBM answers 48 rows read and written at the same time at 5.5 TB/s, but reads alone at 7.0 and writes
// alone at 6.1 to 7.3, so in large launches of larger groups all workgroups of the chip read in one half of a period
// and write in the other.  No workgroup waits for another: each looks at the GPU's constant clock (100 MHz, the same
// on all XCDs) before its loads and before its stores.  In the writing half the classes of workgroups (kCus in a row, which
// work on the same 256 KiB of every row) begin their stores one after the other, each within its part of that half (where the
// arrays lie far apart also within the next one's), and a wave has few stores on their way, so that memory sees almost one row
// at a time.  The first round of the chip waits for nothing, the last not before its stores.  Which
// launches go out so, with which period and what that gives, is at phases_of_launch().
//
// The wait ends when the clock is in [from, from + length) of the period, and after so many looks in any case.
constexpr int kPhaseLooks = 4096;
__device__ __forceinline__ void wait_for_phase(uint32_t per_tick, uint32_t from, uint32_t length) {
  __builtin_amdgcn_sched_barrier(0);
  for (int i = 0; i < kPhaseLooks; ++i) {
    if (static_cast<uint32_t>(__builtin_amdgcn_s_memrealtime()) * per_tick - from < length) break;
    __builtin_amdgcn_s_sleep(1);
  }
  __builtin_amdgcn_sched_barrier(0);
}
struct PhaseGate {
  Phases phases;
  uint32_t at;
  __device__ __forceinline__ explicit PhaseGate(const Phases& p) : phases(p), at(blockIdx.y * p.width + blockIdx.x) {}
  __device__ __forceinline__ void before_loads() const {
    if (at >= phase_round(phases.class_shift)) wait_for_phase(phases.per_tick, 0u, kHalfPeriod);
  }
  __device__ __forceinline__ void before_stores() const {
    if (at >= phase_round(phases.class_shift) && at + phase_round(phases.class_shift) < phases.workgroups)
      wait_for_phase(phases.per_tick, store_phase(at, phases.class_shift), phases.store_for);
  }
};
// Of a wave's stores, those of three members may be on their way: 16 float members 6.19 TB/s with all 48, 6.33 with nine, 6.32 with
// six; 8 float 6.40, 6.49, 6.48; 4 bf16 6.50, 6.57 (six less than nine).
__device__ __forceinline__ void wait_for_stores() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x0F70 | 9);       // vmcnt(9), nothing else
  __builtin_amdgcn_sched_barrier(0);
}

// Eq. 1-3 and the restart for N members held in registers.
template <int N, typename Tag>
__device__ __forceinline__ void update_members(f4 (&p)[N], f4 (&d)[N],
                                               typename ThetaMem<Tag>::mem (&t)[N],
                                               float alpha, float beta, float gamma, float inv_n) {
  typedef ThetaMem<Tag> TM;
  f4 sum_D = p[0] - TM::widen(t[0]);          // Eq. 1, and the two sums of Eq. 2
  f4 sum_P = p[0];
#pragma unroll
  for (int j = 1; j < N; ++j) {
    const f4 D = p[j] - TM::widen(t[j]);
    sum_D = sum_D + D;
    sum_P = sum_P + p[j];
  }
  const f4 mean_P = sum_P * inv_n;
  const f4 t2 = beta * (sum_D * inv_n);
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const f4 t1 = alpha * d[j];
    const f4 t3 = gamma * (p[j] - mean_P);
    const f4 d_new = (t1 - t2) - t3;          // Eq. 2
    const f4 p_new = p[j] + d_new;            // Eq. 3
    d[j] = d_new;
    p[j] = p_new;
    t[j] = TM::narrow(p_new);                // restart of the fast weights
  }
}

// Which of a lane's four elements its workgroup owns: all of them inside a run, some in the first and
// the last vector of a run.  The other elements are loaded with them (a row is a whole number of
// vectors long) and computed with them, but not stored.
struct Owned {
  int first, last;       // elements [first, last) of the vector
  __device__ __forceinline__ bool any() const { return first < last; }
  __device__ __forceinline__ bool all() const { return first == 0 && last == kVecElems; }
};
__device__ __forceinline__ Owned owned_elements(const Piece& r, int32_t lane) {
  Owned o;
  o.first = r.lo - lane > 0 ? r.lo - lane : 0;
  o.last = r.hi - lane < kVecElems ? r.hi - lane : kVecElems;
  return o;
}
template <typename V, typename E>
__device__ __forceinline__ void store_part(RowPiece<E> row, uint32_t lane, V v, Owned o) {
#pragma unroll
  for (uint32_t e = 0; e < kVecElems; ++e)
    if (static_cast<int>(e) >= o.first && static_cast<int>(e) < o.last) row.store_element(lane + e, v[e]);
}
// Asks for all the arguments at once: where they are first used, each would cost the start-up a round trip of its own.
template <typename Args, int N> __device__ __forceinline__ void ask_for(const Args& a, int32_t (&member)[N]) {
  asm volatile("" :: "s"(a.phi), "s"(a.delta), "s"(a.theta), "s"(a.stride), "s"(a.head.cells), "s"(a.head.first),
               "s"(a.head.num_pieces), "s"(a.head.xcd_run), "s"(a.head.swap), "s"(a.head.cell_shift), "s"(a.head.begin_col), "s"(a.head.end_col),
               "s"(member[0]), "s"(member[N > 1 ? 1 : 0]), "s"(member[N > 2 ? 2 : 0]), "s"(member[N > 3 ? 3 : 0]),
               "s"(member[N > 4 ? 4 : 0]), "s"(member[N > 5 ? 5 : 0]), "s"(member[N > 6 ? 6 : 0]), "s"(member[N > 7 ? 7 : 0]),
               "s"(member[N > 8 ? 8 : 0]), "s"(member[N > 9 ? 9 : 0]), "s"(member[N > 10 ? 10 : 0]), "s"(member[N > 11 ? 11 : 0]),
               "s"(member[N > 12 ? 12 : 0]), "s"(member[N > 13 ? 13 : 0]), "s"(member[N > 14 ? 14 : 0]), "s"(member[N > 15 ? 15 : 0]));
}

// 1 / n as the host rounded it where a launch has one size: beside alpha, beta and gamma it costs no load of its own.  Handed
// down as a value it split theirs in three, and pairs of 1024 small tensors took 124.8 us instead of 124.3.
template <int N, typename Args> __device__ __forceinline__ float inv_n(const Args& a) {
  if constexpr (std::is_same<Args, MixedArgs>::value) return 1.0f / static_cast<float>(N);
  else return a.inv_n;
}

// The step of one piece of a group of N whose members are known, everything in registers.
template <int N, typename Tag, bool NT, typename Args>
__device__ __forceinline__ void step_members(const Args& a, const int32_t (&member)[N], const Piece& tr) {
  typedef ThetaMem<Tag> TM;
  typedef typename TM::elem TElem;
  typedef typename TM::mem TMem;
  const uint32_t lane = threadIdx.x * kVecElems;
  const Owned own = owned_elements(tr, static_cast<int32_t>(lane));
  if (!own.any()) return;
  f4 p[N], d[N];
  TMem t[N];
  // Only the rows' offsets are kept for the stores, two scalar registers each; with all 3 N addresses kept, groups
  // of four and more run out of those.
  float* phi = a.phi;
  float* delta = a.delta;
  TElem* theta = static_cast<TElem*>(a.theta);
  int64_t row[N];
  if constexpr (kPhased<Args>) PhaseGate(a.phases).before_loads();
#pragma unroll
  for (int j = 0; j < N; ++j) {
    row[j] = static_cast<int64_t>(member[j]) * a.stride + tr.base;
    p[j] = RowPiece<float>{phi + row[j]}.template load<NT, f4>(lane);
    t[j] = RowPiece<TElem>{theta + row[j]}.template load<NT, TMem>(lane);
  }
#pragma unroll
  for (int j = 0; j < N; ++j) d[j] = RowPiece<float>{delta + row[j]}.template load<NT, f4>(lane);
  // Every load is asked for before the first result is used, delta last since it is needed last.  Without the line below
  // the compiler asks for the last member's delta when all the others have arrived, to save a few registers: a second
  // round trip for every wave from n = 5 on.  us without / with it, arenas in no cache: n = 8 float 10 MB 6.7 / 5.8, 250 MB
  // 88.8 / 87.2, in runs of 1000 97.9 / 94.4; n = 6 float the same 6.5 / 5.7, 87.0 / 84.8, 106 / 95.7; n = 16 float 30 MB
  // 12.8 / 11.7; n = 8 bf16 250 MB in runs of 1000 103.9 / 99.0; n = 10 float 16 MB 8.6 / 7.6.  Some sizes were faster when half
  // the waves came late: n = 5 bf16 30 MB 12.7 / 13.6, n = 7 float 35 MB 13.4 / 14.2, n = 9 bf16 1500 MB 573 / 590.
  __builtin_amdgcn_sched_barrier(0);
  update_members<N, Tag>(p, d, t, a.alpha, a.beta, a.gamma, inv_n<N>(a));
  if constexpr (kPhased<Args>) {
#pragma unroll
    for (int j = 0; j < N; ++j) asm volatile("" : "+v"(p[j]), "+v"(d[j]), "+v"(t[j]));     // everything has arrived
    PhaseGate(a.phases).before_stores();
  }
  auto store_all = [&](auto policy) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
      // Base and offset are added anew, in each of the branches below: kept from the loads, or formed once for all the
      // branches, the addresses are more than fit the scalar registers.
      int64_t at = row[j];
      asm volatile("" : "+s"(at));
      RowPiece<float>{phi + at}.template store<policy.value>(lane, p[j]);
      RowPiece<float>{delta + at}.template store<policy.value>(lane, d[j]);
      RowPiece<TElem>{theta + at}.template store<policy.value>(lane, t[j]);
      if constexpr (kPhased<Args>) wait_for_stores();
    }
  };
  // A piece that is owned in part leaves its stores in the L2, where those of a vector and of elements beside it become
  // one access to memory.
  uint32_t stores = kStreaming;                 // under knobs
  if constexpr (kInOrder<Args>) stores = a.stores;
  if (NT && tr.whole() && stores != kStreaming) {
    if (!kPhased<Args> && stores == kKept) store_all(std::integral_constant<int, kStoreKept>());
    else store_all(std::integral_constant<int, kStoreThrough>());
  } else if (own.all()) {
    store_all(std::integral_constant<int, NT ? kStreamed : kCached>());
  } else {
#pragma unroll
    for (int j = 0; j < N; ++j) {
      int64_t at = row[j];
      asm volatile("" : "+s"(at));
      store_part(RowPiece<float>{phi + at}, lane, p[j], own);
      store_part(RowPiece<float>{delta + at}, lane, d[j], own);
      store_part(RowPiece<TElem>{theta + at}, lane, t[j], own);
    }
  }
}

// Register-resident kernel: group size N known at compile time.
template <int N, typename Tag, bool NT, typename Args>
__global__ void __launch_bounds__(kStepThreads) outer_step_fixed(const Args a) {
  int32_t member[N];
  if constexpr (kInOrder<Args>) {
#pragma unroll
    for (int j = 0; j < N; ++j) member[j] = a.rows[blockIdx.y * N + j];
    ask_for(a, member);
  }
  Piece tr;
  if (!locate(a, tr)) return;
  if constexpr (!kInOrder<Args>) {
#pragma unroll
    for (int j = 0; j < N; ++j) member[j] = a.rows[tr.group * N + j];
  }
  step_members<N, Tag, NT>(a, member, tr);
}

// Groups of different sizes up to MOST in one launch: each workgroup takes the code of its group's size.  A launch of its own
// for every size costs a start and an end each: two pairs and a triple of floats, 1 MB 8.4 -> 5.1 us, 40 MB 18.4 -> 16.5, 200
// MB 67.0 -> 64.9.
template <int MOST, typename Tag>
__global__ void __launch_bounds__(kStepThreads) outer_step_mixed(const MixedArgs a) {
  const uint32_t group = a.groups[blockIdx.y];
  Piece tr;
  if (!locate(a, tr)) return;
  const int32_t* rows = a.rows + (group & 0xFFFFu);
  auto take = [&](auto size) {
    constexpr int N = size.value;
    if constexpr (N <= MOST) {
      int32_t member[N];
#pragma unroll
      for (int j = 0; j < N; ++j) member[j] = rows[j];
      step_members<N, Tag, true>(a, member, tr);
    }
  };
#define NOLOCO_SIZE(N) case N: take(std::integral_constant<int, N>()); break
  switch (group >> 16) {
    NOLOCO_SIZE(1); NOLOCO_SIZE(2); NOLOCO_SIZE(3); NOLOCO_SIZE(4); NOLOCO_SIZE(5); NOLOCO_SIZE(6); NOLOCO_SIZE(7); NOLOCO_SIZE(8);
    NOLOCO_SIZE(9); NOLOCO_SIZE(10); NOLOCO_SIZE(11); NOLOCO_SIZE(12); NOLOCO_SIZE(13); NOLOCO_SIZE(14); NOLOCO_SIZE(15); NOLOCO_SIZE(16);
    default: break;
  }
#undef NOLOCO_SIZE
}

template <typename V, typename E>
__device__ __forceinline__ void store_part(E* p, V v, Owned o) {
#pragma unroll
  for (int e = 0; e < kVecElems; ++e)
    if (e >= o.first && e < o.last) p[e] = v[e];
}
template <bool NT, typename V, typename E>
__device__ __forceinline__ void store_owned(E* p, V v, Owned o) {
  if (o.all()) st<NT>(reinterpret_cast<V*>(p), v);
  else store_part(p, v, o);
}

// Eq. 2-3 and the restart of one member, given the group's two means.
template <typename Tag, bool NT, typename Args>
__device__ __forceinline__ void finish_member(const Args& a, int64_t at, uint32_t lane, f4 p, f4 d, f4 mean_P,
                                              f4 t2, Owned own) {
  typedef ThetaMem<Tag> TM;
  const f4 t1 = a.alpha * d;
  const f4 t3 = a.gamma * (p - mean_P);
  const f4 d_new = (t1 - t2) - t3;
  const f4 p_new = p + d_new;
  store_owned<NT>(a.delta + at + lane, d_new, own);
  store_owned<NT>(a.phi + at + lane, p_new, own);
  store_owned<NT>(static_cast<typename TM::elem*>(a.theta) + at + lane, TM::narrow(p_new), own);
}

// Groups of 17 and more that are not in phases store non-temporally, and outer_step_phi_resident and outer_step_generic have plain
// addresses: with buffers and written-through stores they were up to 4 % faster from 700 MB on, and up to 18 % slower below 60
// MB, where the time a wave takes to form its members' addresses counts.
//
// Subgroups of 17 to 64: too many members to keep phi, delta and theta of all of them in registers,
// but phi alone fits (4 VGPRs per member).  First sweep: load phi and theta of every member, keep
// phi, fold both sums.  Second sweep: load delta, finish, store.  Every byte is still moved once.
// A kernel serves the eight sizes up to NMAX: its last eight members are there while they are below
// n, the same for the whole launch, so the tests are scalar branches.
//
// The two largest leave one wave a SIMD and fetch eight members ahead, so that one wave alone keeps HBM
// busier: n = 64, arenas in no cache, us: bf16 32 MB 30.7 -> 24.6, 96 MB 45.9 -> 40.0, 192 MB 93.4 -> 86.8, 256 MB
// 106.2 -> 103.6; float 32 MB 36.2 -> 28.8, 96 MB 43.2 -> 35.4; 6 and 7 GB within 1 %.  Up to 48, where more
// waves share a SIMD, that is too much in flight (n = 32 float 192 MB 70.6 -> 73.9, n = 24 bf16 400 MB 155.6 ->
// 161.1; n = 48 float 7 GB 2843 -> 2876).
template <int NMAX, typename Tag, bool NT, typename Args>
__global__ void __launch_bounds__(kStepThreads) outer_step_phi_resident(const Args a) {
  constexpr int kChunk = 8;
  typedef ThetaMem<Tag> TM;
  typedef typename TM::elem TElem;
  typedef typename TM::mem TMem;
  Piece tr;
  if (!locate(a, tr)) return;
  const int n = a.n;
  const int32_t* rows = a.rows + tr.group * n;
  const uint32_t lane = threadIdx.x * kVecElems;
  const Owned own = owned_elements(tr, static_cast<int32_t>(lane));
  if (!own.any()) return;
  const TElem* const theta = static_cast<const TElem*>(a.theta);
  auto row = [&](int j) { return static_cast<int64_t>(rows[j]) * a.stride + tr.base; };
  auto there = [&](int j) { return j < NMAX - kChunk || j < n; };
  f4 p[NMAX];
  f4 sum_D, sum_P;
  constexpr bool kAhead = NMAX >= 56;
  TMem t[kAhead ? 2 : 1][kChunk];
  auto fetch = [&](int j0, int buffer) {
#pragma unroll
    for (int k = 0; k < kChunk; ++k)
      if (there(j0 + k)) {
        p[j0 + k] = ld<NT>(reinterpret_cast<const f4*>(a.phi + row(j0 + k) + lane));
        t[buffer][k] = ld<NT>(reinterpret_cast<const TMem*>(theta + row(j0 + k) + lane));
      }
  };
  if constexpr (kAhead) fetch(0, 0);
#pragma unroll
  for (int j0 = 0; j0 < NMAX; j0 += kChunk) {
    const int buffer = kAhead ? j0 / kChunk % 2 : 0;
    if constexpr (kAhead) {
      if (j0 + kChunk < NMAX) fetch(j0 + kChunk, 1 - buffer);
      __builtin_amdgcn_sched_barrier(0);
    } else {
      fetch(j0, 0);
    }
#pragma unroll
    for (int k = 0; k < kChunk; ++k)
      if (there(j0 + k)) {
        const f4 D = p[j0 + k] - TM::widen(t[buffer][k]);
        if (j0 + k == 0) { sum_D = D; sum_P = p[0]; }
        else { sum_D = sum_D + D; sum_P = sum_P + p[j0 + k]; }
      }
    // The sums are formed here and the loads after the next chunk's issued after that: with all of them
    // issued first there is no room for phi.
    asm volatile("" : "+v"(sum_D), "+v"(sum_P) : : "memory");
  }
  const f4 mean_P = sum_P * a.inv_n;
  const f4 t2 = a.beta * (sum_D * a.inv_n);
  f4 d[kAhead ? 2 : 1][kChunk];
  // A lane offset of its own for every chunk: otherwise the addresses of the first sweep are kept for
  // this one, two registers for each of them, and spill.
  uint32_t lane_again = lane;
  auto fetch_delta = [&](int j0, int buffer) {
#pragma unroll
    for (int k = 0; k < kChunk; ++k)
      if (there(j0 + k)) d[buffer][k] = ld<NT>(reinterpret_cast<const f4*>(a.delta + row(j0 + k) + lane_again));
  };
  asm volatile("" : "+v"(lane_again));
  if constexpr (kAhead) fetch_delta(0, 0);
#pragma unroll
  for (int j0 = 0; j0 < NMAX; j0 += kChunk) {
    const int buffer = kAhead ? j0 / kChunk % 2 : 0;
    asm volatile("" : "+v"(lane_again));
    if constexpr (kAhead) {
      if (j0 + kChunk < NMAX) fetch_delta(j0 + kChunk, 1 - buffer);
      __builtin_amdgcn_sched_barrier(0);
    } else {
      fetch_delta(j0, 0);
    }
#pragma unroll
    for (int k = 0; k < kChunk; ++k)
      if (there(j0 + k))
        finish_member<Tag, NT>(a, row(j0 + k), lane_again, p[j0 + k], d[buffer][k], mean_P, t2, own);
    asm volatile("" ::: "memory");
  }
}

// Subgroups of 17 to 56 with phi and delta of every member in registers (eight a member and lane, up to 448 of the 512 that
// one wave a SIMD has); theta goes into the sums as it comes.  Launches in phases need that, since they read in one half of
// the period; there the results are formed between the stores, before the wait they spill from n = 41 on.
// Up to 48 members launches of one wave a SIMD gain by it too, where a second sweep that waits for delta is a round trip more
// for everyone (they take the streaming stores of the kernel above).  us, that kernel / this one, arenas in no cache:
//   n = 17 float 5 MB 10.9 / 9.5  30 MB 16.6 / 13.6    bf16 5 MB 11.7 / 10.6  30 MB 16.4 / 13.3
//   n = 24 float 5 MB 14.3 / 12.2  64 MB 27.4 / 24.7   bf16 5 MB 14.1 / 12.8  52 MB 24.4 / 21.5
//   n = 32 float 30 MB 21.7 / 17.4  100 MB 39.3 / 36.6 bf16 30 MB 23.3 / 19.4  64 MB 30.2 / 28.5
//   n = 48 float 30 MB 29.5 / 25.1  150 MB 59.7 / 56.5 bf16 30 MB 26.1 / 24.2  100 MB 45.6 / 45.4
// The members' ids are read once, for the loads and the stores, and are more than the scalar registers take beside the addresses:
// up to 76 registers move to lanes of vector registers and back (launches in phases from n = 17 on, the others from 25 on), some of
// them between the stores.  Reading the ids again where they are used spares that and is slower: in phases, 1 GB, n = 17 float 334.7 us /
// 338.7, n = 24 361.1 / 365.4, n = 40 361.9 / 368.3, n = 48 bf16 359.6 / 364.2, 6 GB, n = 48 float 1997 / 2032, else the same within 0.5 %;
// short launches, n = 24 float 5 MB 8.31 / 8.63, n = 40 bf16 30 MB 14.4 / 15.0, n = 48 100 MB 39.2 / 39.8.
// With more waves than SIMDs it loses (n = 24 float 80 MB 33.0 / 35.2, n = 32 150 MB 58.7 / 64.1), and so do larger groups, whose
// kernel above fetches ahead (n = 56 float 5 MB 23.6 / 26.4).
constexpr int kHeldMost = 48;
template <int NMAX, typename Tag, typename Args>
__global__ void __launch_bounds__(kStepThreads) outer_step_held(const Args a) {
  constexpr int kChunk = 8, kLast = 8;
  typedef ThetaMem<Tag> TM;
  typedef typename TM::elem TElem;
  typedef typename TM::mem TMem;
  const int n = a.n;
  int32_t member[NMAX];
#pragma unroll
  for (int j = 0; j < NMAX; ++j) {
    const int at = static_cast<int>(blockIdx.y) * n + j;
    member[j] = a.rows[j < NMAX - kLast || at < NOLOCO_MAX_GROUP ? at : NOLOCO_MAX_GROUP - 1];
  }
  ask_for(a, member);
  Piece tr;
  if (!locate(a, tr)) return;
  const uint32_t lane = threadIdx.x * kVecElems;
  const Owned own = owned_elements(tr, static_cast<int32_t>(lane));
  if (!own.any()) return;
  auto there = [&](int j) { return j < NMAX - kLast || j < n; };
  // A row's address is formed anew wherever it is used: 3 NMAX of them are more than fit the scalar registers.
  auto row = [&](int j) {
    int64_t at = static_cast<int64_t>(member[j]) * a.stride + tr.base;
    asm volatile("" : "+s"(at));
    return at;
  };
  const TElem* const theta = static_cast<const TElem*>(a.theta);
  f4 p[NMAX], d[NMAX];
  f4 sum_D, sum_P;
  if constexpr (kPhased<Args>) PhaseGate(a.phases).before_loads();
#pragma unroll
  for (int j0 = 0; j0 < NMAX; j0 += kChunk) {
    TMem t[kChunk];
#pragma unroll
    for (int k = 0; k < kChunk; ++k)
      if (there(j0 + k)) {
        const int64_t at = row(j0 + k);
        p[j0 + k] = RowPiece<float>{a.phi + at}.template load<true, f4>(lane);
        t[k] = RowPiece<const TElem>{theta + at}.template load<true, TMem>(lane);
      }
#pragma unroll
    for (int k = 0; k < kChunk; ++k)
      if (there(j0 + k)) d[j0 + k] = RowPiece<float>{a.delta + row(j0 + k)}.template load<true, f4>(lane);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < kChunk; ++k)
      if (there(j0 + k)) {
        const f4 D = p[j0 + k] - TM::widen(t[k]);
        if (j0 + k == 0) { sum_D = D; sum_P = p[0]; }
        else { sum_D = sum_D + D; sum_P = sum_P + p[j0 + k]; }
      }
    asm volatile("" : "+v"(sum_D), "+v"(sum_P) : : "memory");
  }
  const f4 mean_P = sum_P * a.inv_n;
  const f4 t2 = a.beta * (sum_D * a.inv_n);
  if constexpr (kPhased<Args>) PhaseGate(a.phases).before_stores();
  const bool through = kPhased<Args> && tr.whole();
#pragma unroll
  for (int j = 0; j < NMAX; ++j)
    if (there(j)) {
      const f4 t1 = a.alpha * d[j];
      const f4 t3 = a.gamma * (p[j] - mean_P);
      const f4 d_new = (t1 - t2) - t3;
      const f4 p_new = p[j] + d_new;
      const int64_t at = row(j);
      const RowPiece<float> to_phi{a.phi + at}, to_delta{a.delta + at};
      const RowPiece<TElem> to_theta{static_cast<TElem*>(a.theta) + at};
      if (through) {
        to_phi.template store<kStoreThrough>(lane, p_new);
        to_delta.template store<kStoreThrough>(lane, d_new);
        to_theta.template store<kStoreThrough>(lane, TM::narrow_at_once(p_new));
        if constexpr (kPhased<Args>) wait_for_stores();
      } else if (own.all()) {
        to_phi.template store<kStreamed>(lane, p_new);
        to_delta.template store<kStreamed>(lane, d_new);
        to_theta.template store<kStreamed>(lane, TM::narrow_at_once(p_new));
      } else {
        store_part(to_phi, lane, p_new, own);
        store_part(to_delta, lane, d_new, own);
        store_part(to_theta, lane, TM::narrow_at_once(p_new), own);
      }
    }
}

// Two passes over the members for groups of more than 64: the first forms the two sums, the second
// re-reads phi, reads delta and writes.  Members are taken four at a time with their loads issued
// together; the sums still run strictly in ascending member order.
template <typename Tag, bool NT, typename Args>
__global__ void __launch_bounds__(kStepThreads) outer_step_generic(const Args a) {
  typedef ThetaMem<Tag> TM;
  typedef typename TM::elem TElem;
  typedef typename TM::mem TMem;
  constexpr int kChunk = 4;
  Piece tr;
  if (!locate(a, tr)) return;
  const int n = a.n;
  const int32_t* rows = a.rows + tr.group * n;
  const uint32_t lane = threadIdx.x * kVecElems;
  const Owned own = owned_elements(tr, static_cast<int32_t>(lane));
  if (!own.any()) return;
  const TElem* const theta = static_cast<const TElem*>(a.theta);
  auto row = [&](int j) { return static_cast<int64_t>(rows[j]) * a.stride + tr.base; };
  int64_t at = row(0);
  f4 sum_P = *reinterpret_cast<const f4*>(a.phi + at + lane);            // ordinary loads of phi: read again below
  f4 sum_D = sum_P - TM::widen(ld<NT>(reinterpret_cast<const TMem*>(theta + at + lane)));
  int j = 1;
  for (; j + kChunk <= n; j += kChunk) {
    f4 p[kChunk];
    TMem t[kChunk];
#pragma unroll
    for (int k = 0; k < kChunk; ++k) {
      at = row(j + k);
      p[k] = *reinterpret_cast<const f4*>(a.phi + at + lane);
      t[k] = ld<NT>(reinterpret_cast<const TMem*>(theta + at + lane));
    }
#pragma unroll
    for (int k = 0; k < kChunk; ++k) {
      sum_D = sum_D + (p[k] - TM::widen(t[k]));
      sum_P = sum_P + p[k];
    }
  }
  for (; j < n; ++j) {
    at = row(j);
    const f4 p = *reinterpret_cast<const f4*>(a.phi + at + lane);
    sum_D = sum_D + (p - TM::widen(ld<NT>(reinterpret_cast<const TMem*>(theta + at + lane))));
    sum_P = sum_P + p;
  }
  const f4 mean_P = sum_P * a.inv_n;
  const f4 t2 = a.beta * (sum_D * a.inv_n);
  j = 0;
  for (; j + kChunk <= n; j += kChunk) {
    f4 p[kChunk], d[kChunk];
    int64_t where[kChunk];
#pragma unroll
    for (int k = 0; k < kChunk; ++k) {
      where[k] = row(j + k);
      p[k] = ld<NT>(reinterpret_cast<const f4*>(a.phi + where[k] + lane));
      d[k] = ld<NT>(reinterpret_cast<const f4*>(a.delta + where[k] + lane));
    }
#pragma unroll
    for (int k = 0; k < kChunk; ++k) finish_member<Tag, NT>(a, where[k], lane, p[k], d[k], mean_P, t2, own);
  }
  for (; j < n; ++j) {
    at = row(j);
    finish_member<Tag, NT>(a, at, lane, ld<NT>(reinterpret_cast<const f4*>(a.phi + at + lane)),
                           ld<NT>(reinterpret_cast<const f4*>(a.delta + at + lane)), mean_P, t2, own);
  }
}

// Plain streaming copy: 4 vectors per thread, loads before stores.
__global__ void __launch_bounds__(kBlockThreads) copy_probe_kernel(f4* __restrict__ dst,
                                                                   const f4* __restrict__ src,
                                                                   int64_t vectors) {
  const int64_t first = static_cast<int64_t>(blockIdx.x) * (kBlockThreads * 4) + threadIdx.x;
  f4 v[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t i = first + u * kBlockThreads;
    if (i < vectors) v[u] = __builtin_nontemporal_load(src + i);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t i = first + u * kBlockThreads;
    if (i < vectors) __builtin_nontemporal_store(v[u], dst + i);
  }
}

// Read-only and write-only counterparts of the copy probe (same grid shape).  The read probe
// folds what it loads into a value that is stored only if it equals a pattern the data never
// produces, so the loads cannot be optimised away and nothing is written.
__global__ void __launch_bounds__(kBlockThreads) read_probe_kernel(const f4* __restrict__ src,
                                                                   int64_t vectors, float* sink) {
  const int64_t first = static_cast<int64_t>(blockIdx.x) * (kBlockThreads * 4) + threadIdx.x;
  f4 acc = {0.f, 0.f, 0.f, 0.f};
  f4 v[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t i = first + u * kBlockThreads;
    v[u] = i < vectors ? __builtin_nontemporal_load(src + i) : acc;
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) acc = acc + v[u];
  if (acc.x == 1.2345e-30f && acc.y == -5.4321e-30f) *sink = acc.z;
}

__global__ void __launch_bounds__(kBlockThreads) fill_probe_kernel(f4* __restrict__ dst,
                                                                   int64_t vectors, float value) {
  const int64_t first = static_cast<int64_t>(blockIdx.x) * (kBlockThreads * 4) + threadIdx.x;
  const f4 v = {value, value, value, value};
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int64_t i = first + u * kBlockThreads;
    if (i < vectors) __builtin_nontemporal_store(v, dst + i);
  }
}

// ---------------------------------------------------------------------------------------
// Replica spread (results section of the paper: standard deviation of the weights across the
// data-parallel replicas).  Read-only pass: per column the population variance over the W
// rows in binary32 (sum in ascending row order, mean = sum * inv_W, then the squared
// deviations summed in the same order, times inv_W), pooled in binary64 per tile in a fixed
// order; one small kernel then pools tiles per tensor and tensors overall and takes the roots.
// Bound by HBM reads (7.0 TB/s is what a plain read reaches), so the rows are read once and held, few enough at a time
// for HBM to keep its locality (see spread_run_shift() and spread_workgroups_per_cu()): 8 float rows of 4 GB take 562 us
// (7.1 TB/s) instead of 592 without either, those of the 125M model 579 to 588 (608), 12 of 1024 ragged tensors in 4 M
// elements 36 (37.5).
// ---------------------------------------------------------------------------------------

__device__ __forceinline__ double wave_sum_fixed(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_down(v, off, 64);
  return v;                                   // lane 0 holds the total
}

// The value is the same in every thread.
template <int THREADS> __device__ __forceinline__ double block_sum_fixed(double v, double* wave_part) {
  const double w = wave_sum_fixed(v);
  if ((threadIdx.x & 63) == 0) wave_part[threadIdx.x >> 6] = w;
  __syncthreads();
  double total = wave_part[0];
#pragma unroll
  for (int i = 1; i < THREADS / 64; ++i) total += wave_part[i];
  return total;
}

template <typename Tag> struct SpreadRow;
template <> struct SpreadRow<float> {
  typedef f4 raw;
  static __device__ __forceinline__ f4 widen(f4 v) { return v; }
  static __device__ __forceinline__ void forget_widened(f4&) {}
};
template <> struct SpreadRow<Bf16Tag> {
  typedef u2 raw;                             // four bf16 bit patterns
  static __device__ __forceinline__ f4 widen(u2 v) {
    const u4 w = {v.x << 16, v.x & 0xFFFF0000u, v.y << 16, v.y & 0xFFFF0000u};
    return __builtin_bit_cast(f4, w);
  }
  static __device__ __forceinline__ void forget_widened(u2& v) { asm volatile("" : "+v"(v)); }
};

// What a thread reads: its vector of the columns [base, base + columns) of a row, or zeros where `offset`, its vector's
// from there, is not among them (below 0 is a very large offset).  The memory's bounds check sees to that, so that a
// tensor's edges take no branch and no lane reads what lies beyond them.
struct SpreadColumns {
  int64_t base;          // the same for the whole wave
  int32_t columns;
  int32_t offset;
};
template <int POLICY, typename Tag>
__device__ __forceinline__ typename SpreadRow<Tag>::raw spread_row(const typename ThetaMem<Tag>::elem* at, SpreadColumns c) {
  typedef typename ThetaMem<Tag>::elem TElem;
  typedef typename SpreadRow<Tag>::raw Raw;
  const __amdgpu_buffer_rsrc_t row = buffer_of(at, c.columns * static_cast<int32_t>(sizeof(TElem)));
  const int32_t offset = c.offset * static_cast<int32_t>(sizeof(TElem));
  if constexpr (sizeof(Raw) == 16) return __builtin_bit_cast(Raw, __builtin_amdgcn_raw_buffer_load_b128(row, offset, 0, POLICY));
  else return __builtin_bit_cast(Raw, __builtin_amdgcn_raw_buffer_load_b64(row, offset, 0, POLICY));
}

// A lane's four columns of every row, held in registers as they are stored (a bf16 row takes two registers, not
// four).  Rows 0 .. FULL-1 always exist; rows FULL .. WT-1 exist while they are below W, which is the same for the
// whole launch, so the tests are scalar branches.
template <int WT, int FULL, typename Tag>
__device__ __forceinline__ void load_rows(const SpreadArgs& a, SpreadColumns c, typename SpreadRow<Tag>::raw (&r)[WT]) {
  const typename ThetaMem<Tag>::elem* at = static_cast<const typename ThetaMem<Tag>::elem*>(a.x) + c.base;
#pragma unroll
  for (int w = 0; w < WT; ++w) {
    if (w < FULL || w < a.W) r[w] = spread_row<kStreamed, Tag>(at, c);
    int64_t stride = a.stride;
    if constexpr (WT > 16) asm volatile("" : "+s"(stride));      // one row's address after the other: all at once are more than fit
    at += stride;
  }
}

// Their column variance.
template <int WT, int FULL, typename Tag>
__device__ __forceinline__ f4 column_variance_regs(const SpreadArgs& a, typename SpreadRow<Tag>::raw (&r)[WT]) {
  f4 sum = SpreadRow<Tag>::widen(r[0]);
#pragma unroll
  for (int w = 1; w < WT; ++w)
    if (w < FULL || w < a.W) sum = sum + SpreadRow<Tag>::widen(r[w]);
  const f4 mean = sum * a.inv_W;
  // Without this the compiler keeps the widened rows of the first loop for the second one: 256
  // registers for 64 bf16 rows, which spill (measured 3.0 TB/s against 7.0).  Up to 16 rows there is room for
  // them.
  if constexpr (WT > 16) {
#pragma unroll
    for (int w = 0; w < WT; ++w) SpreadRow<Tag>::forget_widened(r[w]);
  }
  const f4 d0 = SpreadRow<Tag>::widen(r[0]) - mean;
  f4 q = d0 * d0;
#pragma unroll
  for (int w = 1; w < WT; ++w)
    if (w < FULL || w < a.W) {
      const f4 dev = SpreadRow<Tag>::widen(r[w]) - mean;
      q = q + dev * dev;
    }
  return q * a.inv_W;
}

// Any W: two sweeps over memory, four rows at a time.
template <typename Tag>
__device__ __forceinline__ f4 column_variance_mem(const SpreadArgs& a, SpreadColumns c) {
  const typename ThetaMem<Tag>::elem* at = static_cast<const typename ThetaMem<Tag>::elem*>(a.x) + c.base;
  auto row = [&](int w) { return SpreadRow<Tag>::widen(spread_row<kCached, Tag>(at + w * a.stride, c)); };
  f4 sum = row(0);
  int w = 1;
  for (; w + 4 <= a.W; w += 4) {
    const f4 r0 = row(w), r1 = row(w + 1), r2 = row(w + 2), r3 = row(w + 3);
    sum = sum + r0; sum = sum + r1; sum = sum + r2; sum = sum + r3;
  }
  for (; w < a.W; ++w) sum = sum + row(w);
  const f4 mean = sum * a.inv_W;
  const f4 d0 = row(0) - mean;
  f4 q = d0 * d0;
  w = 1;
  for (; w + 4 <= a.W; w += 4) {
    const f4 r0 = row(w) - mean, r1 = row(w + 1) - mean, r2 = row(w + 2) - mean, r3 = row(w + 3) - mean;
    q = q + r0 * r0; q = q + r1 * r1; q = q + r2 * r2; q = q + r3 * r3;
  }
  for (; w < a.W; ++w) {
    const f4 dev = row(w) - mean;
    q = q + dev * dev;
  }
  return q * a.inv_W;
}

// Sum of a lane's four values in binary64, those of columns [lo, hi) only; the first of them is column `column`.
__device__ __forceinline__ double sum_owned(f4 v, int32_t column, int32_t lo, int32_t hi) {
  const float e0 = column + 0 >= lo && column + 0 < hi ? v.x : 0.f;
  const float e1 = column + 1 >= lo && column + 1 < hi ? v.y : 0.f;
  const float e2 = column + 2 >= lo && column + 2 < hi ? v.z : 0.f;
  const float e3 = column + 3 >= lo && column + 3 < hi ? v.w : 0.f;
  return ((static_cast<double>(e0) + static_cast<double>(e1)) + static_cast<double>(e2)) + static_cast<double>(e3);
}

// Vectors per thread: 64 bytes a thread where four vectors make that many (32 of one bf16 row).  A workgroup covers 1024
// columns at a time whatever that is, with one vector per thread where there are enough rows (W = 4 bf16, 400 MB, four
// vectors 62 us, one 56; W = 8 float, 4 GB, 585 / 560), with fewer threads else (W = 2 bf16, 4 GB, one vector per thread 676,
// two 550).
template <int WT, typename Tag> constexpr int kRowBytes = WT * static_cast<int>(sizeof(typename SpreadRow<Tag>::raw));
template <int WT, typename Tag, int STEPS> constexpr int kSpreadVectors =
    WT == 0 || STEPS > 1 ? 1 : kRowBytes<WT, Tag> >= 64 ? 1 : kRowBytes<WT, Tag> >= 32 ? 2 : 4;

// WT = 0 selects the any-W routine.  A workgroup finds its tile with one line of the table of cells, as the step does: by
// binary search over 1024 tensors, 4 M columns x 12 float rows took 31.4 us.  A tile is STEPS times 1024 columns.  Two
// rows are so little for a workgroup that starting them is what counts: large arenas of W = 2 take four steps, all
// loaded together (bf16, 4 GB, 4096 tensors, 593 us with one step and 128 threads, 563 with four).
template <int WT, int FULL, int STEPS, typename Tag>
__global__ void __launch_bounds__((kBlockThreads / kSpreadVectors<WT, Tag, STEPS>)) replica_spread_tiles(const SpreadArgs a) {
  constexpr int U = kSpreadVectors<WT, Tag, STEPS>, kThreads = kBlockThreads / U, kTile = STEPS * kSpreadColumns;
  __shared__ double wave_part[kThreads / 64];
  asm volatile("" :: "s"(a.x), "s"(a.stride), "s"(a.cells), "s"(a.cell_shift), "s"(a.W), "s"(a.inv_W), "s"(a.tiles), "s"(a.run_shift), "s"(a.partials));
  const uint32_t tile = tile_of_block(blockIdx.x, a.run_shift);
  if (tile >= a.tiles) return;
  Piece p;
  locate_by_cells(scalar_pointer(a.cells), a.cell_shift, scalar_pointer(a.spans), static_cast<int64_t>(tile), p, kTile);
  // Step `at` of the tile: the tensor's columns of it, those of a thread's u-th vector, and what that vector reads.
  auto lo_of = [&](int32_t at) { return p.lo > at ? p.lo - at : 0; };
  auto hi_of = [&](int32_t at) { return p.hi < at + kSpreadColumns ? p.hi - at : kSpreadColumns; };
  auto column_of = [&](int32_t u) { return (u * kThreads + static_cast<int32_t>(threadIdx.x)) * kVecElems; };
  auto columns_of = [&](int32_t at, int32_t u) {
    const int32_t first = lo_of(at) / kVecElems * kVecElems, beyond = (hi_of(at) + kVecElems - 1) / kVecElems * kVecElems;   // inside the row
    return SpreadColumns{p.base + at + first, beyond > first ? beyond - first : 0, column_of(u) - first};
  };
  bool any = false;
#pragma unroll
  for (int u = 0; u < U; ++u) any = any || (column_of(u) + kVecElems > p.lo && column_of(u) < p.hi);
  double mine = 0.0;
  if (STEPS > 1 || __ballot(any) != 0) {        // a wave without a column of the tensor has nothing to wait for
    if constexpr (WT > 0) {
      typename SpreadRow<Tag>::raw r[STEPS * U][WT];
#pragma unroll
      for (int i = 0; i < STEPS * U; ++i) load_rows<WT, FULL, Tag>(a, columns_of(i / U * kSpreadColumns, i % U), r[i]);
      // All of them before the first sum.  Without this the compiler takes the steps one after the other, and asks for the last
      // of 64 rows when the others have arrived: 4 GB, us without / with it, W = 64 float 627 / 593, W = 2 bf16 in 65 536 tensors
      // 702 / 638, in 4096 573 / 563.  One step of up to 16 float rows is left alone: of fourteen and sixteen the last one is asked for
      // late too, which paces them further (4 GB 562 / 578 and 559 / 574; with two workgroups a CU 553 and 570, but 287 / 298 and
      // 287 / 294 for 2 GB in 4096 tensors).
      if constexpr (WT > 16 || STEPS > 1 || std::is_same<Tag, Bf16Tag>::value) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < STEPS * U; ++i) {
        const int32_t at = i / U * kSpreadColumns;
        mine += sum_owned(column_variance_regs<WT, FULL, Tag>(a, r[i]), column_of(i % U), lo_of(at), hi_of(at));
      }
    } else {
      mine = sum_owned(column_variance_mem<Tag>(a, columns_of(0, 0)), column_of(0), lo_of(0), hi_of(0));
    }
  }
  const double total = block_sum_fixed<kThreads>(mine, wave_part);
  if (threadIdx.x == 0) {
    a.partials[tile] = total;
    if (tile == 0) *a.ticket = 0;               // for the pooling kernel, which starts after this one
  }
}

// Sum of v[0], v[step], ... below `count` items by one wave, in a fixed order; the value is lane 0's.
// Eight loads per lane are in flight: the sums are latency-bound (65 536 tile sums of one tensor took
// one workgroup with one load in flight per thread 67 us).
__device__ __forceinline__ double wave_pool(const double* v, int64_t count, int64_t step) {
  const int lane = threadIdx.x & 63;
  double acc = 0.0;
  int64_t i = lane;
  for (; i + 7 * 64 < count; i += 8 * 64) {
    double x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = v[(i + k * 64) * step];
#pragma unroll
    for (int k = 0; k < 8; ++k) acc += x[k];
  }
  for (; i < count; i += 64) acc += v[i * step];
  return wave_sum_fixed(acc);
}

// Pools the tile sums: per tensor, then overall.  A workgroup takes one job, see PoolJob: a chunk of a
// long tensor, whose sum replaces the chunk's first tile sum, a whole tensor, or a batch of short ones,
// eight lanes each.  The workgroup that ends last (a ticket, zeroed by the tile kernel) adds up the
// chunks of the long tensors and all tensors, so that everything is pooled in one launch: 1024 tensors
// in 5.2 us, one of 65 536 tiles in 7.4 (a launch per step of it took 4.8 + 4.5 and 67 + 4.6 us).
// Every sum has a fixed order, whichever workgroup is the last.
__global__ void __launch_bounds__(kBlockThreads) replica_spread_pool(const SpreadArgs a, const SegmentTiles* seg,
                                                                     int32_t num_segments, double* out_std) {
  __shared__ double wave_part[kBlockThreads / 64];
  __shared__ uint32_t arrived;
  double* const seg_sums = a.partials + a.tiles;   // per-segment sums are staged behind the tile sums
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  auto finish_segment = [&](int64_t s, int64_t numel, double total) {
    seg_sums[s] = total;
    out_std[s] = numel > 0 ? sqrt(total / static_cast<double>(numel)) : 0.0;
  };
  for (int32_t j = static_cast<int32_t>(blockIdx.x); j < a.num_jobs; j += static_cast<int32_t>(gridDim.x)) {
    const PoolJob job = a.jobs[j];
    if (job.kind == PoolJob::kChunk || job.kind == PoolJob::kWhole) {
      SegmentTiles st = {job.first, job.count, 0};
      if (job.kind == PoolJob::kWhole) st = seg[job.first];
      double acc = 0.0;
      for (int64_t t = threadIdx.x; t < st.num_tiles; t += 8 * kBlockThreads) {
        double x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
          x[k] = t + k * kBlockThreads < st.num_tiles ? a.partials[st.first_tile + t + k * kBlockThreads] : 0.0;
#pragma unroll
        for (int k = 0; k < 8; ++k) acc += x[k];
      }
      const double total = block_sum_fixed<kBlockThreads>(acc, wave_part);   // its barrier: every load above is done
      if (threadIdx.x == 0) {
        if (job.kind == PoolJob::kWhole) finish_segment(job.first, st.numel, total);
        else a.partials[job.first] = total;
      }
      __syncthreads();                                        // wave_part is free for the next job
      continue;
    }
    const int64_t end = job.first + job.count;
    const int64_t longest = job.kind == PoolJob::kBatch ? kPoolChunk : kPoolShort;
    for (int64_t s0 = job.first + wave * kPoolLanes; s0 < end; s0 += kPoolSegments) {
      const int64_t s = s0 + lane / kPoolLanes;
      SegmentTiles st = {0, 0, 0};
      if (s < end) st = seg[s];
      const bool brief = st.num_tiles <= kPoolShort;
      double acc = 0.0;
#pragma unroll
      for (int k = 0; k < kPoolLanes; ++k) {
        const int64_t t = lane % kPoolLanes + k * kPoolLanes;
        if (brief && t < st.num_tiles) acc += a.partials[st.first_tile + t];
      }
#pragma unroll
      for (int off = kPoolLanes / 2; off >= 1; off >>= 1) acc += __shfl_down(acc, off, kPoolLanes);
      const bool first_lane = lane % kPoolLanes == 0;
      if (first_lane && s < end && brief) finish_segment(s, st.numel, acc);
      unsigned long long left = __ballot(first_lane && !brief && st.num_tiles <= longest);
      while (left != 0) {
        const int64_t s_long = s0 + (__ffsll(left) - 1) / kPoolLanes;
        left &= left - 1;
        const double total = wave_pool(a.partials + seg[s_long].first_tile, seg[s_long].num_tiles, 1);
        if (lane == 0) finish_segment(s_long, seg[s_long].numel, total);
      }
    }
  }
  // This workgroup's sums before its ticket.  A barrier does not wait for stores, and the ticket's release
  // waits for those of the wave that draws it: every wave waits for its own first.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (gridDim.x > 1) {
    if (threadIdx.x == 0) arrived = __hip_atomic_fetch_add(a.ticket, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (arrived != gridDim.x - 1) return;
  }
  for (int32_t b = wave; b < a.num_long; b += kBlockThreads / 64) {
    const int64_t s = a.long_segments[b];
    const double total = wave_pool(a.partials + seg[s].first_tile, (seg[s].num_tiles + kPoolChunk - 1) / kPoolChunk, kPoolChunk);
    if (lane == 0) finish_segment(s, seg[s].numel, total);
  }
  __syncthreads();
  double acc = 0.0;
  for (int32_t s = threadIdx.x; s < num_segments; s += kBlockThreads) acc += seg_sums[s];
  const double total = block_sum_fixed<kBlockThreads>(acc, wave_part);
  if (threadIdx.x == 0) out_std[num_segments] = a.elements > 0.0 ? sqrt(total / a.elements) : 0.0;
}

template <int WT, int FULL, int STEPS, typename Tag>
hipError_t enqueue_spread(const SpreadArgs& a, hipStream_t s) {
  const uint32_t round = kXcds << a.run_shift;
  const dim3 grid((a.tiles + round - 1) / round * round), block(kBlockThreads / kSpreadVectors<WT, Tag, STEPS>);
  const int32_t k = spread_workgroups_per_cu(a.W, std::is_same<Tag, Bf16Tag>::value, a.tiles, static_cast<int64_t>(a.elements), a.tile_elems);
  // (64 bytes less than the claim: the workgroup's own)
  return enqueue(replica_spread_tiles<WT, FULL, STEPS, Tag>, grid, block, k != 0 ? lds_for_waves(k) - 64u : 0u, s, a);
}

// Rows in registers for every W up to 64: a kernel of its own up to 16, above that one per eight rows
// whose last eight are conditional.  Larger W sweep memory twice.
template <typename Tag>
hipError_t launch_spread_for_dtype(const SpreadArgs& a, hipStream_t s) {
  if (a.tile_elems != kSpreadColumns) {
    switch (a.W) {
      case 2: return enqueue_spread<2, 2, 4, Tag>(a, s);
      case 4: return enqueue_spread<4, 4, 4, Tag>(a, s);
      case 8: return enqueue_spread<8, 8, 4, Tag>(a, s);
      default: return hipErrorInvalidValue;
    }
  }
  switch (a.W) {
    case 1: return enqueue_spread<1, 1, 1, Tag>(a, s);
    case 2: return enqueue_spread<2, 2, 1, Tag>(a, s);
    case 3: return enqueue_spread<3, 3, 1, Tag>(a, s);
    case 4: return enqueue_spread<4, 4, 1, Tag>(a, s);
    case 5: return enqueue_spread<5, 5, 1, Tag>(a, s);
    case 6: return enqueue_spread<6, 6, 1, Tag>(a, s);
    case 7: return enqueue_spread<7, 7, 1, Tag>(a, s);
    case 8: return enqueue_spread<8, 8, 1, Tag>(a, s);
    case 9: return enqueue_spread<9, 9, 1, Tag>(a, s);
    case 10: return enqueue_spread<10, 10, 1, Tag>(a, s);
    case 11: return enqueue_spread<11, 11, 1, Tag>(a, s);
    case 12: return enqueue_spread<12, 12, 1, Tag>(a, s);
    case 13: return enqueue_spread<13, 13, 1, Tag>(a, s);
    case 14: return enqueue_spread<14, 14, 1, Tag>(a, s);
    case 15: return enqueue_spread<15, 15, 1, Tag>(a, s);
    case 16: return enqueue_spread<16, 16, 1, Tag>(a, s);
    default: break;
  }
  if (a.W <= 24) return enqueue_spread<24, 16, 1, Tag>(a, s);
  if (a.W <= 32) return a.W == 32 ? enqueue_spread<32, 32, 1, Tag>(a, s) : enqueue_spread<32, 24, 1, Tag>(a, s);
  if (a.W <= 40) return enqueue_spread<40, 32, 1, Tag>(a, s);
  if (a.W <= 48) return enqueue_spread<48, 40, 1, Tag>(a, s);
  if (a.W <= 56) return enqueue_spread<56, 48, 1, Tag>(a, s);
  if (a.W <= 64) return a.W == 64 ? enqueue_spread<64, 64, 1, Tag>(a, s) : enqueue_spread<64, 56, 1, Tag>(a, s);
  return enqueue_spread<0, 0, 1, Tag>(a, s);
}

template <typename Tag, bool NT, typename Args>
hipError_t launch_fixed(const Args& args, dim3 grid, uint32_t lds, hipStream_t s) {
  const dim3 block(kStepThreads);
#define NOLOCO_FIXED(N) case N: \
    if constexpr (!kPhased<Args> || N >= kPhasedLeast) return enqueue(outer_step_fixed<N, Tag, NT, Args>, grid, block, lds, s, args); \
    else return hipErrorInvalidValue
  switch (args.n) {
    NOLOCO_FIXED(1); NOLOCO_FIXED(2); NOLOCO_FIXED(3); NOLOCO_FIXED(4);
    NOLOCO_FIXED(5); NOLOCO_FIXED(6); NOLOCO_FIXED(7); NOLOCO_FIXED(8);
    NOLOCO_FIXED(9); NOLOCO_FIXED(10); NOLOCO_FIXED(11); NOLOCO_FIXED(12);
    NOLOCO_FIXED(13); NOLOCO_FIXED(14); NOLOCO_FIXED(15); NOLOCO_FIXED(16);
    default: return hipErrorInvalidValue;
  }
#undef NOLOCO_FIXED
}

template <typename Tag, bool NT, typename Args>
hipError_t launch_for_size(const Args& args, dim3 grid, uint32_t lds, hipStream_t s) {
  const dim3 block(kStepThreads);
#define NOLOCO_RESIDENT(N) return enqueue(outer_step_phi_resident<N, Tag, NT, Args>, grid, block, lds, s, args)
  if (args.n <= 16) return launch_fixed<Tag, NT>(args, grid, lds, s);
  if (args.n <= 24) NOLOCO_RESIDENT(24);
  if (args.n <= 32) NOLOCO_RESIDENT(32);
  if (args.n <= 40) NOLOCO_RESIDENT(40);
  if (args.n <= 48) NOLOCO_RESIDENT(48);
  if (args.n <= 56) NOLOCO_RESIDENT(56);
  if (args.n <= 64) NOLOCO_RESIDENT(64);
  return enqueue(outer_step_generic<Tag, NT, Args>, grid, block, lds, s, args);
#undef NOLOCO_RESIDENT
}

template <int ROWS> InOrderArgs<ROWS> in_order_args(const StepArgs& a, const InOrderHead& head) {
  InOrderArgs<ROWS> args;
  args.phi = a.phi;
  args.delta = a.delta;
  args.theta = a.theta;
  args.stride = a.stride;
  args.head = head;
  args.alpha = a.alpha;
  args.beta = a.beta;
  args.gamma = a.gamma;
  args.inv_n = a.inv_n;
  args.n = a.n;
  args.stores = a.stores;
  std::memcpy(args.rows, a.rows, sizeof(args.rows));
  return args;
}

template <typename Tag, typename Args>
hipError_t launch_held(const Args& args, dim3 grid, uint32_t lds, hipStream_t s) {
  const dim3 block(kStepThreads);
#define NOLOCO_HELD(N) return enqueue(outer_step_held<N, Tag, Args>, grid, block, lds, s, args)
  if (args.n <= 24) NOLOCO_HELD(24);
  if (args.n <= 32) NOLOCO_HELD(32);
  if (args.n <= 40) NOLOCO_HELD(40);
  if (args.n <= 48) NOLOCO_HELD(48);
  if constexpr (kPhased<Args>) {
    if (args.n <= kPhasedMost) NOLOCO_HELD(56);
  }
  return hipErrorInvalidValue;
#undef NOLOCO_HELD
}

// A launch in phases has waves and an order of its own: as many as there are classes, the pieces as dealt.
template <typename Tag>
hipError_t launch_phased(const StepArgs& paced, hipStream_t s) {
  StepArgs step = paced;
  step.xcd_run = 1;
  const InOrderHead head = in_order_head(step);
  const uint32_t round = in_order_round(step.xcd_run), lds = lds_for_waves(1 << step.phases.class_shift);
  const dim3 grid((head.num_pieces + round - 1) / round * round, static_cast<uint32_t>(step.num_groups));
  PhasedArgs args;
  static_cast<InOrderArgs<NOLOCO_MAX_GROUP>&>(args) = in_order_args<NOLOCO_MAX_GROUP>(step, head);
  args.phases = step.phases;
  args.phases.width = grid.x;
  args.phases.workgroups = grid.x * grid.y;
  return args.n <= 16 ? launch_fixed<Tag, true>(args, grid, lds, s) : launch_held<Tag>(args, grid, lds, s);
}

template <typename Tag>
hipError_t launch_for_dtype(const StepArgs& args, const KernelChoice& choice, hipStream_t s) {
  if (choice.in_order != 0) {
    if (args.phases.per_tick != 0) return launch_phased<Tag>(args, s);
    const InOrderHead head = in_order_head(args);
    const uint32_t round = in_order_round(args.xcd_run);
    const dim3 grid((head.num_pieces + round - 1) / round * round, static_cast<uint32_t>(args.num_groups));
    if (args.n <= 16 && args.n * args.num_groups <= kFewRows)
      return launch_fixed<Tag, true>(in_order_args<kFewRows>(args, head), grid, choice.lds, s);
    const auto in_order = in_order_args<NOLOCO_MAX_GROUP>(args, head);
    if (args.n > 16 && args.n <= kHeldMost && static_cast<int64_t>(head.num_pieces) * args.num_groups <= 4 * kCus)
      return launch_held<Tag>(in_order, grid, choice.lds, s);
    return launch_for_size<Tag, true>(in_order, grid, choice.lds, s);
  }
  uint32_t wgs = args.work_items << args.piece_shift;
  if (args.xcd_map != 0) {
    const uint32_t run = args.xcd_map == 1 ? 1u : static_cast<uint32_t>(args.xcd_map) << args.piece_shift;
    wgs = (wgs + kXcds * run - 1) / (kXcds * run) * (kXcds * run);
  }
  return choice.nontemporal != 0 ? launch_for_size<Tag, true>(args, dim3(wgs), 0u, s)
                                 : launch_for_size<Tag, false>(args, dim3(wgs), 0u, s);
}

// Adds the groups of one size to those that share a launch, and launches them with the last.
int launch_together(const StepArgs& args, int32_t theta_dtype, const KernelChoice& choice, hipStream_t s) {
  Together& all = *choice.together;
  if (args.n > 16 || all.rows + args.n * args.num_groups > kMixedRows) return static_cast<int>(hipErrorInvalidValue);
  for (int32_t g = 0; g < args.num_groups; ++g)
    all.group[all.groups + g] = static_cast<uint32_t>(all.rows + g * args.n) | static_cast<uint32_t>(args.n) << 16;
  std::memcpy(all.member + all.rows, args.rows, static_cast<size_t>(args.n * args.num_groups) * sizeof(int32_t));
  all.groups += args.num_groups;
  all.rows += args.n * args.num_groups;
  all.most = all.most > args.n ? all.most : args.n;
  if (args.n * args.num_groups > all.usual) {
    all.usual = args.n * args.num_groups;
    all.lds = choice.lds;
  }
  if (!choice.last) return 0;
  StepArgs whole = args, part;
  whole.num_groups = all.groups;
  if (part_of_launch(whole, 0, &part) != whole.num_tiles) return static_cast<int>(hipErrorInvalidValue);
  const InOrderHead head = in_order_head(part);
  const uint32_t round = in_order_round(part.xcd_run);
  const dim3 grid((head.num_pieces + round - 1) / round * round, static_cast<uint32_t>(all.groups)), block(kStepThreads);
  MixedArgs mixed;
  static_cast<InOrderArgs<kMixedRows>&>(mixed) = in_order_args<kMixedRows>(part, head);
  std::memcpy(mixed.rows, all.member, sizeof(mixed.rows));
  std::memcpy(mixed.groups, all.group, sizeof(mixed.groups));
  const bool bf16 = theta_dtype == NOLOCO_BF16;
#define NOLOCO_MIXED(MOST) \
  static_cast<int>(bf16 ? enqueue(outer_step_mixed<MOST, Bf16Tag>, grid, block, all.lds, s, mixed) \
                        : enqueue(outer_step_mixed<MOST, float>, grid, block, all.lds, s, mixed))
  return all.most <= 4 ? NOLOCO_MIXED(4) : all.most <= 8 ? NOLOCO_MIXED(8) : NOLOCO_MIXED(16);
#undef NOLOCO_MIXED
}

// Scratch of noloco_replica_spread_noalloc: tile partial sums, then per-segment sums.  One copy
// per GPU, allocated with the code object and kept until the process ends.  In host code this
// name is only a handle for hipGetSymbolAddress; kernels receive the resolved device address.
static __device__ __align__(256) double spread_scratch[kSpreadScratchDoubles];

constexpr int kMaxDevices = 64;
double* scratch_of_device[kMaxDevices];          // resolved addresses, filled on first use per device
std::atomic<bool> scratch_known[kMaxDevices];

}  // namespace

int launch_outer_step(const StepArgs& args, int32_t theta_dtype, const KernelChoice& choice,
                      void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (args.num_tiles <= 0 || args.num_groups <= 0) return 0;
  if (choice.together != nullptr) return launch_together(args, theta_dtype, choice, s);
  StepArgs part;
  for (int64_t t = 0; t < args.num_tiles;) {
    t += part_of_launch(args, t, &part);
    const hipError_t e = theta_dtype == NOLOCO_BF16 ? launch_for_dtype<Bf16Tag>(part, choice, s)
                                                    : launch_for_dtype<float>(part, choice, s);
    if (e != hipSuccess) return static_cast<int>(e);
  }
  return 0;
}

int launch_replica_spread(const SpreadArgs& asked, int32_t x_dtype, const SegmentTiles* seg_tiles,
                          int32_t num_segments, double* out_std, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  SpreadArgs args = asked;
  if (args.run_shift != 0) args.run_shift = spread_run_shift(args.W, x_dtype == NOLOCO_BF16, args.tiles, args.tile_elems);
  if (args.tiles > 0) {
    const hipError_t e = x_dtype == NOLOCO_BF16 ? launch_spread_for_dtype<Bf16Tag>(args, s)
                                                : launch_spread_for_dtype<float>(args, s);
    if (e != hipSuccess) return static_cast<int>(e);
  }
  // No tile kernel, no zeroed ticket: one workgroup then takes every job.
  const dim3 grid(args.tiles > 0 && args.num_jobs > 1 ? static_cast<uint32_t>(args.num_jobs) : 1u);
  return static_cast<int>(enqueue(replica_spread_pool, grid, dim3(kBlockThreads), 0u, s, args, seg_tiles, num_segments, out_std));
}

int static_spread_scratch(double** out) {
  int device = -1;
  hipError_t e = hipGetDevice(&device);
  if (e != hipSuccess) return static_cast<int>(e);
  if (device < 0 || device >= kMaxDevices) return static_cast<int>(hipErrorInvalidDevice);
  if (!scratch_known[device].load(std::memory_order_acquire)) {
    // Every GPU holds its own copy of the array at its own address: resolve with that GPU current.
    // Two threads racing here resolve the same address twice, which is harmless.
    void* address = nullptr;
    e = hipGetSymbolAddress(&address, HIP_SYMBOL(spread_scratch));
    if (e != hipSuccess) return static_cast<int>(e);
    if (address == nullptr) return static_cast<int>(hipErrorInvalidSymbol);
    scratch_of_device[device] = static_cast<double*>(address);
    scratch_known[device].store(true, std::memory_order_release);
  }
  *out = scratch_of_device[device];
  return 0;
}

int launch_stream_probe(int mode, void* dst, const void* src, int64_t bytes, float value,
                        void* stream) {
  const int64_t vectors = bytes / 16;
  const int64_t per_block = kBlockThreads * 4;
  const int64_t blocks = (vectors + per_block - 1) / per_block;
  if (blocks > kMaxGridWorkgroups) return static_cast<int>(hipErrorInvalidValue);
  const dim3 grid(static_cast<uint32_t>(blocks)), block(kBlockThreads);
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (mode == 0)
    return static_cast<int>(enqueue(copy_probe_kernel, grid, block, 0u, s, static_cast<f4*>(dst),
                                    static_cast<const f4*>(src), vectors));
  if (mode == 1)
    return static_cast<int>(enqueue(read_probe_kernel, grid, block, 0u, s, static_cast<const f4*>(src),
                                    vectors, static_cast<float*>(dst)));
  return static_cast<int>(enqueue(fill_probe_kernel, grid, block, 0u, s, static_cast<f4*>(dst), vectors, value));
}

}  // namespace noloco
