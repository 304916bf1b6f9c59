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
  __attribute__((aligned(16))) int counts[2][kVecs * kWaves], turns[2 * kWaves];
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
    int c[kBatch];
#pragma unroll
    for (int r = 0; r < kBatch; ++r) c[r] = __popcll(m[r]);
#pragma unroll
    for (int d = 1; d < kBatch; d *= 2)  // a tree: a chain of additions waits for each of them
#pragma unroll
      for (int r = 0; r + d < kBatch; r += 2 * d) c[r] += c[r + d];
    n += c[0];
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

// The same from known counts at lo and hi, and only to the value with exactly k above it or the largest with more: two rounds of
// three aim at it along the line between the counts, which halves the rounds (9 to 5 where a third of the keys is to go) and
// costs as much as counting some keys.
template <typename Count>
__device__ __forceinline__ uint32_t bisect_exact(uint32_t lo, uint32_t hi, int n_lo, int n_hi, int k, Count count) {
#pragma unroll 1
  for (int i = 0; n_lo != k && hi - lo > 1u; ++i) {
    uint32_t step = (hi - lo) / 2;
    if (i % 3 != 2) {
      const float part = (float)(n_lo - k) * __builtin_amdgcn_rcpf((float)(n_lo - n_hi));
      step = (uint32_t)((float)(hi - lo) * part);
      step = (uint32_t)__builtin_amdgcn_readfirstlane((int)min(max(step, 1u), hi - lo - 1u));
    }
    const int n = count(lo + step);
    if (n >= k) { lo += step; n_lo = n; }
    else { hi = lo + step; n_hi = n; }
  }
  return lo;
}

// bisect over the keys of a whole workgroup, kN per thread; turns: 2 * waves ints of LDS. All threads call it.
template <int kThreads, int kN>
__device__ __forceinline__ uint32_t bisect_spread(const uint32_t (&v)[kN], uint32_t lo, uint32_t hi, int k, int enough, int* turns) {
  constexpr int kWaves = kThreads / kWave;
  static_assert(kWaves % 4 == 0, "counts are read four at a time");
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  int turn = 0;
  return bisect(lo, hi, k, enough, [&](uint32_t x) {
    const int n = count_above(v, x);
    turn ^= kWaves;  // the counts of one round are read while those of the next are written
    if (lane == 0) turns[turn + wave] = n;
    __syncthreads();
    int sum = 0;
#pragma unroll
    for (int w = 0; w < kWaves; w += 4) {
      const int4 q = *reinterpret_cast<const int4*>(&turns[turn + w]);
      sum += q.x + q.y + q.z + q.w;
    }
    return __builtin_amdgcn_readfirstlane(sum);
  });
}

// The kb largest of a workgroup's keys, of which more than kb lie above `low`, in the order (v, thread, i) of key[kPer * v + i]:
// emit(at, j) once per selected key. above, equal: kVecs * waves ints each, 16-byte aligned, turns as above; all of them unused by
// others since the last barrier. All threads call it.
template <int kThreads, int kVecs, int kPer, typename Emit>
__device__ __forceinline__ void select_spread(const uint32_t (&key)[kVecs * kPer], uint32_t low, uint32_t high, int kb, Emit emit,
                                              int* above, int* equal, int* turns) {
  constexpr int kWaves = kThreads / kWave;
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  // the k-th key, or (exactly kb keys above T - 1) a value that only selected keys reach
  const uint32_t T = bisect_spread<kThreads>(key, low, high, kb, kb, turns) + 1u;
#pragma unroll
  for (int v = 0; v < kVecs; ++v) {
    int n = 0, e = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      n += __popcll(__ballot(key[kPer * v + i] > T));
      e += __popcll(__ballot(key[kPer * v + i] == T));
    }
    if (lane == 0) { above[v * kWaves + wave] = n; equal[v * kWaves + wave] = e; }
  }
  __syncthreads();
  int place[kVecs], ties[kVecs];
  const int need = kb - wave_prefixes<kVecs, kWaves>(above, wave, place);  // keys equal to T that are taken, the first ones
  wave_prefixes<kVecs, kWaves>(equal, wave, ties);
#pragma unroll
  for (int v = 0; v < kVecs; ++v) {
    int sure_b = place[v], tie_b = ties[v];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      sure_b = lanes_before(__ballot(key[kPer * v + i] > T), sure_b);
      tie_b = lanes_before(__ballot(key[kPer * v + i] == T), tie_b);
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int j = kPer * v + i;
      if (key[j] > T) {
        emit(min(tie_b, need) + sure_b++, j);
      } else if (key[j] == T) {
        if (tie_b < need) emit(sure_b + tie_b, j);
        ++tie_b;
      }
    }
  }
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

// The kb largest of `total` <= 64 * kN gathered keys, of which all are above `low` and none above `top`, in page order, by one
// wave: emit(r, at, page) says that the page, which the lane holds as its r-th, is the at-th selected one, or with at = -1 that
// it is none. ahead(page) is called for all kN pages of the lanes (0: none) before the search.
template <int kN, typename Emit, typename Ahead>
__device__ __forceinline__ void select_gathered(const uint2* kept, int total, uint32_t low, uint32_t top, int kb, Emit emit,
                                                Ahead ahead) {
  const int lane = threadIdx.x % kWave;
  uint32_t key[kN];
  int page[kN];
#pragma unroll
  for (int r = 0; r < kN; ++r) {
    const uint2 e = kept[r * kWave + lane];  // (what lies behind the last one is not used)
    key[r] = r * kWave + lane < total ? e.x : 0u;
    page[r] = r * kWave + lane < total ? (int)e.y : 0;
  }
  ahead(page);
  // x with exactly kb keys above it, or the largest x with more: the next value is then the k-th key
  auto count = [&](uint32_t y) { return count_above(key, y); };
  uint32_t x = low;
  if constexpr (kN >= 8) x = bisect_exact(low, top, total, 0, kb, count);
  else if (total > kb) x = bisect(low, top, kb, kb, count);
  int at = 0, ties = 0;
  if (count_above(key, x) == kb) {
#pragma unroll
    for (int r = 0; r < kN; ++r) {
      const bool mine = key[r] > x;
      const unsigned long long sel = __ballot(mine);
      emit(r, mine ? lanes_before(sel, at) : -1, page[r]);
      at += __popcll(sel);
    }
    return;
  }
  const uint32_t T = x + 1u;
  const int need = kb - count_above(key, T);  // keys equal to T that are taken, from the lowest page up
#pragma unroll
  for (int r = 0; r < kN; ++r) {
    const unsigned long long tie = __ballot(key[r] == T);
    const bool mine = key[r] > T || (key[r] == T && lanes_before(tie, ties) < need);
    const unsigned long long sel = __ballot(mine);
    emit(r, mine ? lanes_before(sel, at) : -1, page[r]);
    at += __popcll(sel);
    ties += __popcll(tie);
  }
}
template <int kN, typename Emit>
__device__ __forceinline__ void select_gathered(const uint2* kept, int total, uint32_t low, uint32_t top, int kb, Emit emit) {
  select_gathered<kN>(kept, total, low, top, kb, emit, [](const int(&)[kN]) {});
}

// The kb largest of `total` <= kSmallCap gathered keys, all above `low`, by every wave for itself, with their physical pages from the
// row's page table (of at least one entry), which are looked up while the search runs: emit_all(r, at, page, phys), see
// select_gathered.
template <typename EmitAll>
__device__ __forceinline__ void select_kept(const uint2* kept, int total, uint32_t low, int kb, const int32_t* page_table,
                                            EmitAll emit_all) {
  const int lane = threadIdx.x % kWave;
  auto gathered = [&](auto per_lane) {
    constexpr int kN = decltype(per_lane)::value;
    int phys[kN];
    uint32_t top = 0u;
#pragma unroll
    for (int r = 0; r < kN; ++r) top = max(top, r * kWave + lane < total ? kept[r * kWave + lane].x : 0u);
    top = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_allreduce_minmax<true>(top));
    select_gathered<kN>(kept, total, low, top, kb, [&](int r, int at, int page) { emit_all(r, at, page, phys[r]); },
                        [&](const int(&page)[kN]) {
#pragma unroll
                          for (int r = 0; r < kN; ++r) phys[r] = page_table[page[r]];
                        });
  };
  if (total <= 2 * kWave) gathered(std::integral_constant<int, 2>());
  else if (total <= 4 * kWave) gathered(std::integral_constant<int, 4>());
  else if (total <= 8 * kWave) gathered(std::integral_constant<int, 8>());
  else gathered(std::integral_constant<int, 16>());
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
    select_kept(sh.kept, total, T0 - 1u, kb, page_table, emit_all);
    return;
  }
  if constexpr (kThreads * kVecs * 4 > kSmallCap) {
    // masses of equal scores, or a k beyond the groups: the keys in the registers of all waves
    __syncthreads();  // the counts have been read by all
    select_spread<kThreads, kVecs, 4>(key, T0 - 1u, 0xffffffffu, kb, [&](int at, int j) { emit_own(at, page_of(j)); },
                                      sh.counts[0], sh.counts[1], sh.turns);
    __syncthreads();
  }
}

}  // namespace
}  // namespace unique
