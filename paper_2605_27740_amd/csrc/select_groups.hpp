// Gathering the keys that can be among the k largest of a row from the maxima of its groups of pages: the device code that the
// selection kernel for long rows (select_grouped.hip, which explains it) and the decode step (step.hip) share.
#pragma once
#include "select_small.hpp"

namespace unique {
namespace {

template <int kThreads, int kVecs, int kCap>
struct GroupShared {
  static constexpr int kWaves = kThreads / kWave;
  static constexpr int kMaxGroups = kVecs * kThreads / 2;  // kept groups: two 16-byte loads of scores each
  static constexpr int kCounts = kVecs * kWaves;
  uint32_t wave_min[kWaves], wave_max[kWaves];
  __attribute__((aligned(16))) int counts[2][kCounts], turns[2 * kWaves];
  int group_list[kMaxGroups + kWave];  // the last ones are for lanes without a group
  uint2 kept[kCap + kWave];            // key, page
};

// A row's gathered keys: `total` of them, at most kCap, all from T0 on and fewer than kb above top, in sh.kept in page order.
struct Gathered {
  uint32_t T0, top;
  int total;
};

// 0 < kb < P, kb at most kCap and 8/9 of kMaxGroups; pages from forced_from on, at most kb, are always selected. All threads call
// it; ends with a barrier.
template <int kThreads, int kGroupVecs, int kVecs, int kCap>
__device__ __forceinline__ Gathered gather_from_groups(const float* srow, const uint32_t* grow, int P, int kb, int forced_from,
                                                       GroupShared<kThreads, kVecs, kCap>& sh) {
  constexpr int kWaves = kThreads / kWave, kMaxGroups = GroupShared<kThreads, kVecs, kCap>::kMaxGroups;
  static_assert(kGroupVecs <= kVecs, "the counts hold either");
  const int t = threadIdx.x, lane = t % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const int groups = (P + kGroupPages - 1) / kGroupPages;
  auto& counts = sh.counts;
  uint32_t key[4 * kVecs];
  int first[kVecs];  // the first page of every four keys

  // ---- 1. T0, a value that at least kb groups reach
  uint32_t gkey[4 * kGroupVecs], top = 0u, least = 0xffffffffu;
  auto group_of = [&](int j) { return row_page<kThreads, 4>(j); };
  {
    // the last page of a row may have been scored apart from its group, whose maximum then does not count it
    const uint32_t last = score_key(srow[P - 1]);
    const bool alone = P % kGroupPages == 1;
    uint4 raw[kGroupVecs];
#pragma unroll
    for (int v = 0; v < kGroupVecs; ++v) {
      raw[v] = make_uint4(0u, 0u, 0u, 0u);
      if (group_of(4 * v) < groups) raw[v] = *reinterpret_cast<const uint4*>(grow + group_of(4 * v));
    }
#pragma unroll
    for (int j = 0; j < 4 * kGroupVecs; ++j) {
      uint32_t k = j % 4 == 0 ? raw[j / 4].x : (j % 4 == 1 ? raw[j / 4].y : (j % 4 == 2 ? raw[j / 4].z : raw[j / 4].w));
      const int g = group_of(j);
      if (g == groups - 1) k = alone ? last : max(k, last);
      gkey[j] = g >= groups ? 0u : (forced_from < P && (g + 1) * kGroupPages > forced_from ? kKeyForced : k);
      top = max(top, g < groups ? k : 0u);  // (of scores alone, see search_top)
      least = min(least, g < groups ? gkey[j] : 0xffffffffu);
    }
  }
  // Every wave finds a bound that its share of kb of its own groups reaches; the smallest bound then has kb groups. That costs
  // a fifth more groups than a bound over all of them, and no barrier per round, where the scores do not depend on the position.
  uint32_t T0 = 1u;
  top = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_allreduce_minmax<true>(top));
  {
    uint32_t mine = 0xffffffffu;
    int of_wave = 0;
#pragma unroll
    for (int j = 0; j < 4 * kGroupVecs; ++j) of_wave += __popcll(__ballot(gkey[j] > 0u));
    // a wave with few groups has a poor bound, which the others do without
    constexpr int kFull = 4 * kWave;
    const int rest = groups % kFull, without = groups - rest;
    const bool drop = groups < 4 * kThreads && rest < kFull / 2 && kb <= without;
    const int counted = drop ? without : groups;
    if (kb <= groups && of_wave > 0 && !(drop && of_wave < kFull)) {  // uniform
      least = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_allreduce_minmax<false>(least));
      const int share = (int)(((int64_t)kb * of_wave + counted - 1) / counted);
      const uint32_t high = forced_from < P ? search_top(gkey, share) : top;
      mine = bisect(least - 1u, high, of_wave, share, share + share / 8, [&](uint32_t x) { return count_above(gkey, x); }) + 1u;
    }
    if (lane == 0) { sh.wave_max[wave] = top; sh.wave_min[wave] = mine; }
    __syncthreads();
    uint32_t low = 0xffffffffu;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) { top = max(top, sh.wave_max[w]); low = min(low, sh.wave_min[w]); }
    if (kb <= groups) T0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)low);
    top = P - forced_from < kb ? (uint32_t)__builtin_amdgcn_readfirstlane((int)top) : kKeyForced;
  }

  // ---- 2. the groups from T0 on, in page order
  int place[kVecs], gplace[kGroupVecs];
  int kept_groups = place_from<kThreads, kGroupVecs, 4>(gkey, T0, counts[0], gplace);
  // Scores that rise or fall along the row give the waves poor bounds (several times kb groups), and many groups may be equal, of
  // which the first are enough: each holds a key that equals the bound. Quotas of more waves leave more, so their number counts.
  // A step of 8192 pages, k = 256, so / with rows that have too many groups read again: rising by two standard deviations
  // 28.2 / 60.9 us, five values 29.2 / 109; 32768 pages, five values 44 / 378. Groups dealt to the waves in turn, so that their
  // shares are alike, cost scores without an order 0.5 to 1 us and left the rising ones where they are. The code for it is kept out
  // of the way of the others (16 x 8192 pages, nothing in the caches: 53.7 us in line, 52.8 so).
  if (__builtin_expect(kept_groups > min(kb + kb / 2 + 12 * kWaves, kMaxGroups), 0)) {  // uniform
    T0 = tighten<kThreads, kGroupVecs, 4>(gkey, T0, top, kept_groups, kb, kb + kb / 8, counts[1], sh.turns);
    kept_groups = place_from<kThreads, kGroupVecs, 4>(gkey, T0, counts[0], gplace);
  }
#pragma unroll
  for (int v = 0; v < kGroupVecs; ++v) {
    int at = gplace[v];
#pragma unroll
    for (int i = 0; i < 4; ++i) at = lanes_before(__ballot(gkey[4 * v + i] >= T0), at);
#pragma unroll
    for (int i = 0; i < 4; ++i) {  // without branches: they cost more than the stores that they save
      const bool in = gkey[4 * v + i] >= T0;
      sh.group_list[in ? at : kMaxGroups + lane] = group_of(4 * v + i);
      at += in;
    }
  }
  __syncthreads();

  // ---- 3. their scores: load (v, thread) is the half (thread % 2) of a group, so the pages ascend with (v, thread)
  const int loads = (2 * kept_groups + kThreads - 1) / kThreads;  // loads that any thread has
  {
    float4 raw[kVecs];
#pragma unroll
    for (int v = 0; v < kVecs; ++v) {
      const int at = (v * kThreads + t) / 2;
      first[v] = at < kept_groups ? sh.group_list[at] * kGroupPages + (t % 2) * 4 : P;
      raw[v] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (first[v] < P) raw[v] = *reinterpret_cast<const float4*>(srow + first[v]);  // the row is padded to a multiple of 64
    }
#pragma unroll
    for (int v = 0; v < kVecs; ++v) {
      key[4 * v] = key[4 * v + 1] = key[4 * v + 2] = key[4 * v + 3] = 0u;
      if (v >= loads) continue;  // uniform, here and below
      keys_of(raw[v], P - first[v], key + 4 * v);
      if (forced_from < P) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (first[v] + i >= forced_from && first[v] + i < P) key[4 * v + i] = kKeyForced;
      }
    }
  }

  // ---- 4. those from T0 on are gathered, in page order
  int total = place_from<kThreads, kVecs, 4>(key, T0, counts[1], place, loads);
  if (__builtin_expect(total > kCap, 0)) {  // uniform
    T0 = tighten<kThreads, kVecs, 4>(key, T0, top, total, kb, (kb + kCap) / 2, counts[0], sh.turns);
    total = place_from<kThreads, kVecs, 4>(key, T0, counts[1], place, loads);
  }
#pragma unroll
  for (int v = 0; v < kVecs; ++v) {
    if (v >= loads) break;
    int at = place[v];
#pragma unroll
    for (int i = 0; i < 4; ++i) at = lanes_before(__ballot(key[4 * v + i] >= T0), at);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool in = key[4 * v + i] >= T0;
      sh.kept[in ? at : kCap + lane] = make_uint2(key[4 * v + i], (uint32_t)(first[v] + i));
      at += in;
    }
  }
  __syncthreads();
  return {T0, top, total};
}

}  // namespace
}  // namespace unique
