// The selection of the top-k pages of a row by a small workgroup with the row's keys in registers, for rows of a few thousand
// pages (select.hip has the kernels for longer ones, and explains what is selected).
//
// One workgroup is bound by the instructions that it spends per key and by its barriers. So every key is looked at as little
// as possible: a lower bound T0 of the k-th key comes from the maxima of disjoint groups of keys (the k-th largest maximum
// is one: k groups reach it), found by bisection in registers; the keys from T0 on -- about k and a third more -- are gathered
// in the LDS in page order, and every wave bisects for the exact k-th of them by itself. Three barriers, and no atomics.
#pragma once
#include <type_traits>

#include "select_core.hpp"

namespace unique {
namespace {

constexpr int kSmallCap = 1024;  // gathered keys: 16 per lane of a wave

template <int kThreads, int kVecs>
struct SmallShared {
  static constexpr int kWaves = kThreads / kWave;
  uint32_t group_max[kThreads * kVecs];
  __attribute__((aligned(16))) int counts[2][kVecs * kWaves];
  __attribute__((aligned(16))) uint2 kept[kSmallCap + kWave];  // key, page; the last ones are for lanes without a key
};

// Number of the wave's values above x, kN per lane. The comparisons are all made before the first result is counted: left to
// itself the compiler sends them through one register pair, and every one waits for the one before.
template <int kN>
__device__ __forceinline__ int count_above(const uint32_t (&v)[kN], uint32_t x) {
  constexpr int kBatch = kN < 8 ? kN : 8;
  int n = 0;
#pragma unroll
  for (int r0 = 0; r0 < kN; r0 += kBatch) {
    unsigned long long m[kBatch];
#pragma unroll
    for (int r = 0; r < kBatch; ++r) m[r] = __ballot(v[r0 + r] > x);
    if constexpr (kBatch == 2) asm volatile("" : "+s"(m[0]), "+s"(m[1]));
    if constexpr (kBatch == 4) asm volatile("" : "+s"(m[0]), "+s"(m[1]), "+s"(m[2]), "+s"(m[3]));
    if constexpr (kBatch == 8)
      asm volatile("" : "+s"(m[0]), "+s"(m[1]), "+s"(m[2]), "+s"(m[3]), "+s"(m[4]), "+s"(m[5]), "+s"(m[6]), "+s"(m[7]));
#pragma unroll
    for (int r = 0; r < kBatch; ++r) n += __popcll(m[r]);
  }
  return n;
}

// A value x with count(x) >= k, from lo (count(lo) >= k) and hi (count(hi) < k), where count falls with x: the first one met
// with count(x) <= enough, or the largest such x. At most 32 rounds.
template <typename Count>
__device__ __forceinline__ uint32_t bisect(uint32_t lo, uint32_t hi, int k, int enough, Count count) {
  if (hi - lo <= 1u) return lo;
  bool stop;
#pragma unroll 1
  do {
    const uint32_t mid = lo + (hi - lo) / 2;
    const int n = count(mid);
    lo = n >= k ? mid : lo;
    hi = n >= k ? hi : mid;
    stop = ((n >= k) & (n <= enough)) | (hi - lo <= 1u);
  } while (!stop);
  return lo;
}

// A lower bound (>= 1) of the k-th largest key from n = 64 * kN group maxima, at least k of them above 0: a value that k to
// about 9/8 k groups reach.
template <int kN>
__device__ __forceinline__ uint32_t bound_of_maxima(const uint32_t* group_max, int k) {
  const int lane = threadIdx.x % kWave;
  uint32_t m[kN], top = 0u, least = 0xffffffffu;
#pragma unroll
  for (int r = 0; r < kN; ++r) {
    m[r] = group_max[r * kWave + lane];
    top = max(top, m[r]);
    least = min(least, m[r]);
  }
  top = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_allreduce_minmax<true>(top));
  least = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_allreduce_minmax<false>(least));
  return bisect(least > 0u ? least - 1u : 0u, top, k, k + k / 8, [&](uint32_t x) { return count_above(m, x); }) + 1u;
}

// The kb largest of `total` <= 64 * kN gathered keys, of which all are above `low`, in page order. Every wave finds them all:
// emit(r, at, page, phys) says that the page, which the lane holds as its r-th, is the at-th selected one, or with at = -1
// that it is none. The physical pages are looked up while the search runs.
template <int kN, typename Emit>
__device__ __forceinline__ void select_gathered(const uint2* kept, int total, uint32_t low, int kb, const int32_t* page_table,
                                                Emit emit) {
  const int lane = threadIdx.x % kWave;
  uint32_t key[kN], top = 0u;
  int page[kN], phys[kN];
#pragma unroll
  for (int r = 0; r < kN; ++r) {
    const uint2 e = kept[r * kWave + lane];  // (what lies behind the last one is not used)
    key[r] = r * kWave + lane < total ? e.x : 0u;
    page[r] = r * kWave + lane < total ? (int)e.y : 0;
  }
#pragma unroll
  for (int r = 0; r < kN; ++r) {
    phys[r] = page_table[page[r]];
    top = max(top, key[r]);
  }
  top = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_allreduce_minmax<true>(top));
  // x with exactly kb keys above it, or the largest x with more: the next value is then the k-th key
  uint32_t x = low;
  if (total > kb) x = bisect(low, top, kb, kb, [&](uint32_t y) { return count_above(key, y); });
  const uint32_t T = x + 1u;
  const int need = kb - count_above(key, T);  // keys equal to T that are taken, from the lowest page up
  int at = 0, ties = 0;
#pragma unroll
  for (int r = 0; r < kN; ++r) {
    const unsigned long long tie = __ballot(key[r] == T);
    const bool mine = key[r] > T || (key[r] == T && lanes_before(tie, ties) < need);
    const unsigned long long sel = __ballot(mine);
    emit(r, mine ? lanes_before(sel, at) : -1, page[r], phys[r]);
    at += __popcll(sel);
    ties += __popcll(tie);
  }
}

// Thread t holds the keys of the pages row_page(j) (0: no page); 0 < kb < P; page_table: the row's, of at least one entry.
// emit_all(r, at, page, phys) is called by every wave for all that its lanes hold (see select_gathered); if too many keys are left to
// gather, emit_own(at, page) is called once per selected page instead, followed by a barrier.
template <int kThreads, int kVecs, typename EmitAll, typename EmitOwn>
__device__ __forceinline__ void select_small(const uint32_t (&key)[4 * kVecs], int P, int kb, const int32_t* page_table,
                                             EmitAll emit_all, EmitOwn emit_own, SmallShared<kThreads, kVecs>& sh) {
  constexpr int kWaves = kThreads / kWave;
  const int t = threadIdx.x, lane = t % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
  auto page_of = [](int j) { return row_page<kThreads, 4>(j); };

  // ---- 1. T0: groups are the keys of a thread, or of a half or a quarter of its loads where that makes too few groups.
  // With k near the number of groups T0 would be close to the smallest maximum, which leaves too many keys.
  const int loads = (P + 3) / 4;
  auto enough_groups = [&](int per_thread) { return 8 * kb <= 5 * min(kThreads * per_thread, loads); };
  uint32_t T0 = 1u;
  if (kb <= min(kThreads * kVecs, loads)) {  // uniform
    uint32_t m[kVecs];
#pragma unroll
    for (int v = 0; v < kVecs; ++v)
      m[v] = max(max(key[4 * v], key[4 * v + 1]), max(key[4 * v + 2], key[4 * v + 3]));
    auto bound = [&](auto per_thread) {  // the groups of thread t are its loads v = g, g + per_thread, ...
      constexpr int kPerThread = decltype(per_thread)::value;
#pragma unroll
      for (int g = 0; g < kPerThread; ++g) {
        uint32_t top = m[g];
#pragma unroll
        for (int v = g + kPerThread; v < kVecs; v += kPerThread) top = max(top, m[v]);
        sh.group_max[g * kThreads + t] = top;
      }
      __syncthreads();
      T0 = bound_of_maxima<kPerThread * kWaves>(sh.group_max, kb);
    };
    if (kVecs == 1 || enough_groups(1)) bound(std::integral_constant<int, 1>());
    else if (kVecs == 2 || enough_groups(2)) bound(std::integral_constant<int, kVecs < 2 ? 1 : 2>());
    else bound(std::integral_constant<int, kVecs>());
  }

  // ---- 2. the keys from T0 on, in page order
#pragma unroll
  for (int v = 0; v < kVecs; ++v) {
    int n = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) n += __popcll(__ballot(key[4 * v + i] >= T0));
    if (lane == 0) sh.counts[0][v * kWaves + wave] = n;
  }
  __syncthreads();
  int place[kVecs];
  const int total = wave_prefixes<kVecs, kWaves>(sh.counts[0], wave, place);
  if (total <= kSmallCap) {  // uniform
#pragma unroll
    for (int v = 0; v < kVecs; ++v) {
      int at = place[v];
#pragma unroll
      for (int i = 0; i < 4; ++i) at = lanes_before(__ballot(key[4 * v + i] >= T0), at);
#pragma unroll
      for (int i = 0; i < 4; ++i) {  // without branches: they cost more than the stores that they save
        const bool in = key[4 * v + i] >= T0;
        sh.kept[in ? at : kSmallCap + lane] = make_uint2(key[4 * v + i], (uint32_t)page_of(4 * v + i));
        at += in;
      }
    }
    __syncthreads();
    if (total <= 2 * kWave) select_gathered<2>(sh.kept, total, T0 - 1u, kb, page_table, emit_all);
    else if (total <= 4 * kWave) select_gathered<4>(sh.kept, total, T0 - 1u, kb, page_table, emit_all);
    else if (total <= 8 * kWave) select_gathered<8>(sh.kept, total, T0 - 1u, kb, page_table, emit_all);
    else select_gathered<16>(sh.kept, total, T0 - 1u, kb, page_table, emit_all);
    return;
  }
  if constexpr (kThreads * kVecs * 4 > kSmallCap) {
    // Masses of equal scores, or a k beyond the groups: bisection over the keys in the registers of all waves.
    int turn = 0;
    const uint32_t x = bisect(T0 - 1u, 0xffffffffu, kb, kb, [&](uint32_t y) {
      const int n = count_above(key, y);
      turn ^= 1;
      if (lane == 0) sh.group_max[turn * kWaves + wave] = (uint32_t)n;
      __syncthreads();
      int sum = 0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) sum += (int)sh.group_max[turn * kWaves + w];
      return __builtin_amdgcn_readfirstlane(sum);
    });
    const uint32_t T = x + 1u;  // the k-th key, or (exactly kb keys above x) a value that only selected keys reach
    __syncthreads();            // the counts of the gathering have been read by all
#pragma unroll
    for (int v = 0; v < kVecs; ++v) {
      int n = 0, e = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        n += __popcll(__ballot(key[4 * v + i] > T));
        e += __popcll(__ballot(key[4 * v + i] == T));
      }
      if (lane == 0) { sh.counts[0][v * kWaves + wave] = n; sh.counts[1][v * kWaves + wave] = e; }
    }
    __syncthreads();
    int ties[kVecs];
    const int need = kb - wave_prefixes<kVecs, kWaves>(sh.counts[0], wave, place);
    wave_prefixes<kVecs, kWaves>(sh.counts[1], wave, ties);
#pragma unroll
    for (int v = 0; v < kVecs; ++v) {
      int sure_b = place[v], tie_b = ties[v];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        sure_b = lanes_before(__ballot(key[4 * v + i] > T), sure_b);
        tie_b = lanes_before(__ballot(key[4 * v + i] == T), tie_b);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int j = 4 * v + i;
        if (key[j] > T) {
          emit_own(min(tie_b, need) + sure_b++, page_of(j));
        } else if (key[j] == T) {
          if (tie_b < need) emit_own(sure_b + tie_b, page_of(j));
          ++tie_b;
        }
      }
    }
    __syncthreads();
  }
}

}  // namespace
}  // namespace unique
