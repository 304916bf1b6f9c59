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
  static constexpr int kCounts = (kVecs > kCap / kThreads ? kVecs : kCap / kThreads) * kWaves;
  uint32_t wave_min[kWaves], wave_max[kWaves];
  __attribute__((aligned(16))) int counts[2][kCounts], turns[2 * kWaves];
  int group_list[kMaxGroups + kWave];  // the last ones are for lanes without a group
  uint2 kept[kCap + kWave];            // key, page
};

// A row's gathered keys: `total` of them, all from T0 on and none above top, in sh.kept in page order if they fit; more than
// kCap are left in the registers (key, and the first page of every four), and with more groups than kMaxGroups total is -1.
template <int kVecs>
struct Gathered {
  uint32_t T0, top;
  int total;
  uint32_t key[4 * kVecs];
  int first[kVecs];
};

// 0 < kb < P; pages from forced_from on are always selected. All threads call it; ends with a barrier if the keys are in sh.kept.
template <int kThreads, int kGroupVecs, int kVecs, int kCap>
__device__ __forceinline__ void gather_from_groups(const float* srow, const uint32_t* grow, int P, int kb, int forced_from,
                                                   Gathered<kVecs>& got, GroupShared<kThreads, kVecs, kCap>& sh) {
  constexpr int kWaves = kThreads / kWave, kMaxGroups = GroupShared<kThreads, kVecs, kCap>::kMaxGroups;
  const int t = threadIdx.x, lane = t % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const int groups = (P + kGroupPages - 1) / kGroupPages;
  auto& counts = sh.counts;
  auto& key = got.key;
  auto& first = got.first;

  // ---- 1. T0, a value that at least kb groups reach
  uint32_t gkey[4 * kGroupVecs], top = 0u, least = 0xffffffffu;
  auto group_of = [&](int j) { return row_page<kThreads, 4>(j); };
  {
    uint4 raw[kGroupVecs];
#pragma unroll
    for (int v = 0; v < kGroupVecs; ++v) {
      raw[v] = make_uint4(0u, 0u, 0u, 0u);
      if (group_of(4 * v) < groups) raw[v] = *reinterpret_cast<const uint4*>(grow + group_of(4 * v));
    }
#pragma unroll
    for (int j = 0; j < 4 * kGroupVecs; ++j) {
      const uint32_t k = j % 4 == 0 ? raw[j / 4].x : (j % 4 == 1 ? raw[j / 4].y : (j % 4 == 2 ? raw[j / 4].z : raw[j / 4].w));
      const int g = group_of(j);
      gkey[j] = g >= groups ? 0u : (forced_from < P && (g + 1) * kGroupPages > forced_from ? kKeyForced : k);
      top = max(top, gkey[j]);
      least = min(least, g < groups ? gkey[j] : 0xffffffffu);
    }
  }
  // Every wave finds a bound that its share of kb of its own groups reaches; the smallest bound then has kb groups. That costs
  // a fifth more groups than a bound over all of them and no barrier per round.
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
      mine = bisect(least - 1u, top, share, share + share / 8, [&](uint32_t x) { return count_above(gkey, x); }) + 1u;
    }
    if (lane == 0) { sh.wave_max[wave] = top; sh.wave_min[wave] = mine; }
    __syncthreads();
    uint32_t low = 0xffffffffu;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) { top = max(top, sh.wave_max[w]); low = min(low, sh.wave_min[w]); }
    if (kb <= groups) T0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)low);
    top = (uint32_t)__builtin_amdgcn_readfirstlane((int)top);
  }

  // ---- 2. the groups from T0 on, in page order
  int place[kVecs], gplace[kGroupVecs];
  {
    int(*gcounts) = counts[0];
#pragma unroll
    for (int v = 0; v < kGroupVecs; ++v) {
      int n = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) n += __popcll(__ballot(gkey[4 * v + i] >= T0));
      if (lane == 0) gcounts[v * kWaves + wave] = n;
    }
    __syncthreads();
  }
  const int kept_groups = wave_prefixes<kGroupVecs, kWaves>(counts[0], wave, gplace);
  got.T0 = T0;
  got.top = top;
  got.total = -1;
  if (kept_groups > kMaxGroups) return;  // uniform
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
#pragma unroll
  for (int v = 0; v < kVecs; ++v) {
    int n = 0;
    if (v < loads) {
#pragma unroll
      for (int i = 0; i < 4; ++i) n += __popcll(__ballot(key[4 * v + i] >= T0));
    }
    if (lane == 0) counts[1][v * kWaves + wave] = n;
  }
  __syncthreads();
  const int total = wave_prefixes<kVecs, kWaves>(counts[1], wave, place);
  got.total = total;
  if (total > kCap) return;  // uniform
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

}

// Masses of equal scores, of which more groups reach the bound than are gathered: select by re-reading the row. emit(at, page).
template <int kThreads, typename Emit>
__device__ __forceinline__ void select_by_rereading(const float* srow, int P, int kb, int forced_from, Emit emit,
                                                    SelectShared<kThreads>& sh) {
  constexpr int kWaves = kThreads / kWave;
  const int t = threadIdx.x, lane = t % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
  auto key_of = [&](int page) { return page >= forced_from ? kKeyForced : score_key(srow[page]); };
  uint32_t kmin = 0xffffffffu, kmax = 0u;
  for (int p = t; p < P; p += kThreads) {
    const uint32_t k = key_of(p);
    const bool finite = k > kKeyNegInf && k < kKeyPosInf;
    kmin = min(kmin, finite ? k : 0xffffffffu);
    kmax = max(kmax, finite ? k : 0u);
  }
  kmin = wave_allreduce_minmax<false>(kmin);
  kmax = wave_allreduce_minmax<true>(kmax);
    if (lane == 0) { sh.wave_min[wave] = kmin; sh.wave_max[wave] = kmax; }
  constexpr int kBuckets = SelectShared<kThreads>::kBuckets;
  for (int i = t; i < kBuckets + kBuckets / 4; i += kThreads) sh.hist[i] = 0;
  if (t == 0) sh.ncand = 0;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) { kmin = min(kmin, sh.wave_min[w]); kmax = max(kmax, sh.wave_max[w]); }
  select_reread<kThreads>(key_of, P, kb, bucket_map(kmin, kmax, kBuckets), emit, sh);
}

}  // namespace
}  // namespace unique
