// The selection of the top-k pages of a row by a small workgroup with the row's keys in registers, for rows of a few thousand
// pages (select.hip has the kernels for longer ones, and explains what is selected).
//
// One workgroup is bound by the instructions that it spends per key and by its barriers. So every key is looked at as little
// as possible: a lower bound T0 of the k-th key comes from the maxima of disjoint groups of keys (the k-th largest maximum
// is one: k groups reach it), found by bisection in registers; the keys from T0 on -- about k and a third more -- are gathered
// in the LDS in page order, and every wave bisects for the exact k-th of them by itself. Three barriers, and no atomics. Where more
// keys reach T0 than the LDS has room for (masses of ties), the bound is first made tighter, with a barrier per round.
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
  static_assert((kBatch & (kBatch - 1)) == 0 && kN % kBatch == 0, "whole batches");
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

// A value x with count(x) >= k, from lo (count(lo) = n_lo >= k) and hi (count(hi) < k), where count falls with x: the first one met
// with count(x) <= enough, or the largest x. At most 32 rounds.
template <typename Count>
__device__ __forceinline__ uint32_t bisect(uint32_t lo, uint32_t hi, int n_lo, int k, int enough, Count count) {
#pragma unroll 1
  while ((n_lo > enough) & (hi - lo > 1u)) {
    const uint32_t mid = lo + (hi - lo) / 2;
    const int n = count(mid);
    lo = n >= k ? mid : lo;
    n_lo = n >= k ? n : n_lo;
    hi = n >= k ? hi : mid;
  }
  return lo;
}

// The same from known counts at lo and hi, where two rounds of three aim between k and `enough` along the line between the counts.
// That halves the number of rounds (9 to 5 where a third of the keys is to go) and costs as much as counting some keys. Keys are
// nearly logarithms of the scores, which suits the tail of a distribution; across very many octaves, zero that is, the line is drawn
// between the scores themselves (8192 pages that score -p / 8192, k = 256: 31.1 us with keys alone, 27.3 so). Where most keys are
// equal an aim leaves nearly everything, so there are no more than twelve rounds with aims. Leaves count(x) in n_lo.
template <typename Count>
__device__ __forceinline__ uint32_t bisect_aimed(uint32_t lo, uint32_t hi, int& n_lo, int n_hi, int k, int enough, Count count) {
  constexpr uint32_t kOctaves = 16u << 23;
#pragma unroll 1
  for (int i = 0; (n_lo > enough) & (hi - lo > 1u); ++i) {
    const uint32_t width = hi - lo;
    uint32_t x = lo + width / 2;
    if (i % 3 != 2 && i < 12) {
      const float part = (float)(n_lo - (k + enough) / 2) * __builtin_amdgcn_rcpf((float)(n_lo - n_hi));
      uint32_t aim = lo + (uint32_t)((float)width * part);
      if (width > kOctaves) {
        const float from = ordered_to_float(lo), f = fmaf(ordered_to_float(hi) - from, part, from);
        aim = fabsf(f) < 3.0e38f ? score_key(f) : x;  // infinite or no number: halve
      }
      x = (uint32_t)__builtin_amdgcn_readfirstlane((int)min(max(aim, lo + 1u), hi - 1u));
    }
    const int n = count(x);
    if (n >= k) { lo = x; n_lo = n; }
    else { hi = x; n_hi = n; }
  }
  return lo;
}

// The upper end of a search for the k-th of the wave's values: the largest of them, or, with pages that are always selected (whose
// keys are far above all others), the largest other one if fewer than k lie above it.
template <int kN>
__device__ __forceinline__ uint32_t search_top(const uint32_t (&v)[kN], int k) {
  uint32_t top = 0u;
#pragma unroll
  for (int r = 0; r < kN; ++r) top = max(top, v[r]);
  top = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_allreduce_minmax<true>(top));
  if (top == kKeyForced) {  // uniform
    uint32_t other = 0u;
#pragma unroll
    for (int r = 0; r < kN; ++r) other = max(other, v[r] == kKeyForced ? 0u : v[r]);
    other = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_allreduce_minmax<true>(other));
    if (count_above(v, other) < k) top = other;
  }
  return top;
}

// Number of a workgroup's keys above x, kN per thread; turns: 2 * waves ints of LDS. All threads call it; it holds a barrier.
template <int kThreads, int kN>
struct SpreadCount {
  static constexpr int kWaves = kThreads / kWave;
  static_assert(kWaves % 4 == 0, "counts are read four at a time");
  const uint32_t (&v)[kN];
  int* turns;
  int turn = 0;
  __device__ __forceinline__ int operator()(uint32_t x) {
    const int n = count_above(v, x);
    turn ^= kWaves;  // the counts of one round are read while those of the next are written
    if (threadIdx.x % kWave == 0) turns[turn + threadIdx.x / kWave] = n;
    __syncthreads();
    int sum = 0;
#pragma unroll
    for (int w = 0; w < kWaves; w += 4) {
      const int4 q = *reinterpret_cast<const int4*>(&turns[turn + w]);
      sum += q.x + q.y + q.z + q.w;
    }
    return __builtin_amdgcn_readfirstlane(sum);
  }
};

// A bound T0 that `total` > enough >= kb of a workgroup's keys reach, of which fewer than kb are above `top`, is raised until at most
// `enough` reach it. Where so many are equal that no bound leaves between kb and `enough`, the first of them, in the order (v, thread,
// i) of key[kPer * v + i], are left that make kb, and the others become 0: of equal keys the first are selected. equal: kVecs * waves
// ints, 16-byte aligned, turns as above; both unused by others since the last barrier. All threads call it; it holds barriers.
template <int kThreads, int kVecs, int kPer>
__device__ __forceinline__ uint32_t tighten(uint32_t (&key)[kVecs * kPer], uint32_t T0, uint32_t top, int total, int kb, int enough,
                                            int* equal, int* turns) {
  constexpr int kWaves = kThreads / kWave;
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  SpreadCount<kThreads, kVecs * kPer> count{key, turns};
  // T0 is often the key that masses of others equal
  const int above = count(T0);
  uint32_t T = T0;
  int n = total;
  if (above >= kb) {
    n = above;
    T = bisect_aimed(T0, top, n, 0, kb, enough, [&](uint32_t x) { return count(x); }) + 1u;
  }
  if (n <= enough) return T;  // uniform
#pragma unroll
  for (int v = 0; v < kVecs; ++v) {
    int e = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) e += __popcll(__ballot(key[kPer * v + i] == T));
    if (lane == 0) equal[v * kWaves + wave] = e;
  }
  __syncthreads();
  int ties[kVecs];
  const int rest = kb - n + wave_prefixes<kVecs, kWaves>(equal, wave, ties);  // how many of the equal ones are left
#pragma unroll
  for (int v = 0; v < kVecs; ++v) {
    int tie = ties[v];
#pragma unroll
    for (int i = 0; i < kPer; ++i) tie = lanes_before(__ballot(key[kPer * v + i] == T), tie);
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const bool is = key[kPer * v + i] == T;
      if (is && tie >= rest) key[kPer * v + i] = 0u;
      tie += is;
    }
  }
  return T;
}

// counts[v * waves + wave] = keys from T0 on, of the wave's with that v; a barrier; their prefixes (see wave_prefixes) and their total.
// The keys with v >= used (uniform) are all 0.
template <int kThreads, int kVecs, int kPer>
__device__ __forceinline__ int place_from(const uint32_t (&key)[kVecs * kPer], uint32_t T0, int* counts, int (&place)[kVecs],
                                          int used = kVecs) {
  constexpr int kWaves = kThreads / kWave;
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
#pragma unroll
  for (int v = 0; v < kVecs; ++v) {
    int n = 0;
    if (v < used) {
#pragma unroll
      for (int i = 0; i < kPer; ++i) n += __popcll(__ballot(key[kPer * v + i] >= T0));
    }
    if (lane == 0) counts[v * kWaves + wave] = n;
  }
  __syncthreads();
  return wave_prefixes<kVecs, kWaves>(counts, wave, place);
}

// A lower bound (>= 1) of the k-th largest key from 64 * kN group maxima, `groups` >= k of them above 0: a value that k to about
// 9/8 k groups reach. (All, if there are no more: 80 x 32 pages, k = 8, in one kernel 23.7 us with a search, 21.4 so.)
template <int kN>
__device__ __forceinline__ uint32_t bound_of_maxima(const uint32_t* group_max, int groups, int k) {
  const int lane = threadIdx.x % kWave;
  uint32_t m[kN], least = 0xffffffffu;
#pragma unroll
  for (int r = 0; r < kN; ++r) {
    m[r] = group_max[r * kWave + lane];
    least = min(least, m[r] - 1u);  // (0, no key, wraps around)
  }
  least = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_allreduce_minmax<false>(least));
  return bisect(least, search_top(m, k), groups, k, k + k / 8, [&](uint32_t x) { return count_above(m, x); }) + 1u;
}

// The kb largest of `total` <= 64 * kN gathered keys, of which all are above `low` and fewer than kb above `top`, in page order, by one
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
  int n = total;
  const int above = total > 2 * kb ? count(low + 1u) : kb;  // so many only if many equal the first one
  if (above < kb) top = low + 1u;
  if constexpr (kN >= 8) x = bisect_aimed(low, top, n, 0, kb, kb, count);
  else { x = bisect(low, top, total, kb, kb, count); n = count(x); }
  int at = 0, ties = 0;
  if (n == kb) {
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
    uint32_t key[kN];
#pragma unroll
    for (int r = 0; r < kN; ++r) key[r] = r * kWave + lane < total ? kept[r * kWave + lane].x : 0u;
    const uint32_t top = search_top(key, kb);
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

// Thread t holds the keys of the pages row_page(j) (0: no page), which may be changed; 0 < kb < P, kb at most half of kSmallCap;
// page_table: the row's, of at least one entry. emit_all(r, at, page, phys) is called by every wave for all that its lanes hold
// (see select_gathered).
template <int kThreads, int kVecs, typename EmitAll>
__device__ __forceinline__ void select_small(uint32_t (&key)[4 * kVecs], int P, int kb, const int32_t* page_table,
                                             EmitAll emit_all, SmallShared<kThreads, kVecs>& sh) {
  constexpr int kWaves = kThreads / kWave;
  const int t = threadIdx.x, lane = t % kWave;
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
      T0 = bound_of_maxima<kPerThread * kWaves>(sh.group_max, min(kThreads * kPerThread, loads), kb);
    };
    if (kVecs == 1 || enough_groups(1)) bound(std::integral_constant<int, 1>());
    else if (kVecs == 2 || enough_groups(2)) bound(std::integral_constant<int, kVecs < 2 ? 1 : 2>());
    else bound(std::integral_constant<int, kVecs>());
  }

  // ---- 2. the keys from T0 on, in page order
  int place[kVecs];
  int total = place_from<kThreads, kVecs, 4>(key, T0, sh.counts[0], place);
  if constexpr (kThreads * kVecs * 4 > kSmallCap) {
    if (__builtin_expect(total > kSmallCap, 0)) {  // uniform: masses of equal scores, or a k beyond the groups
      T0 = tighten<kThreads, kVecs, 4>(key, T0, kKeyForced, total, kb, kSmallCap / 2, sh.counts[1], sh.turns);
      total = place_from<kThreads, kVecs, 4>(key, T0, sh.counts[0], place);
    }
  }
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
}

}  // namespace
}  // namespace unique
