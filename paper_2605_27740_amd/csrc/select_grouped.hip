// Top-k selection for long rows whose group maxima the score kernel has left beside the scores (one key per 8 pages).
//
// A row belongs to one workgroup, whose loads bound the selection of a long row: 62501 scores are 250 KB for one compute unit,
// read twice. Here the maxima are read instead. At least k groups reach the k-th largest of them, T0, so the k-th score does,
// too, and only the groups that reach T0 -- about k -- can hold a selected page: their scores alone are read, an eighth of the
// row plus 8 k of them. T0 and then the exact k-th key
// are found by bisection over keys in registers.
// One wave makes the last step, whose rounds would need barriers of all the others.
// What bounds it is a chain of such steps on one compute unit, of 30 900 cycles for 62501 pages, k = 1024: maxima 3900, T0 5600,
// list of the groups 2300, their scores 5300, gathering 3800, the k-th key 6400, the output 3000.
#include <algorithm>
#include <type_traits>

#include "select_small.hpp"

namespace unique {
namespace {

// kGroupVecs: 16-byte loads of group maxima per thread.
template <int kThreads, int kGroupVecs>
__global__ __launch_bounds__(kThreads) void topk_select_grouped_kernel(CacheView c, const float* __restrict__ scores,
                                                                       const uint32_t* __restrict__ group_max,
                                                                       int score_stride, int top_k,
                                                                       int32_t* __restrict__ sel_pages,
                                                                       int32_t* __restrict__ sel_count) {
  constexpr int kWaves = kThreads / kWave;
  constexpr int kVecs = 8;                            // 16-byte loads of scores per thread
  constexpr int kMaxGroups = kVecs * kThreads / 2;    // kept groups: two loads each
  constexpr int kKept = 4096;                         // keys from T0 on
  __shared__ SelectShared<kThreads> sh;
  __shared__ __attribute__((aligned(16))) int counts[2][(kVecs > kKept / kThreads ? kVecs : kKept / kThreads) * kWaves], turns[2 * kWaves];
  __shared__ int group_list[kMaxGroups + kWave];  // the last ones are for lanes without a group
  __shared__ uint2 kept[kKept + kWave];  // key, page

  const int row = blockIdx.x;
  const int b = row / c.Hkv;
  const int t = threadIdx.x, lane = t % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const int N = c.seq_lens[b];
  int P = min((N + c.S - 1) / c.S, c.max_pages_hint);
  P = min(P, kThreads * kGroupVecs * 4 * kGroupPages);  // a row longer than the host bound is cut, never overrun
  const int kb = min(top_k, P);
  int32_t* out = sel_pages + (int64_t)row * top_k;
  const float* srow = scores + (int64_t)row * score_stride;
  const int group_stride = score_stride / kGroupPages;  // a multiple of 8
  const uint32_t* grow = group_max + (int64_t)row * group_stride;

  for (int i = kb + t; i < top_k; i += kThreads) out[i] = -1;
  if (t == 0) sel_count[row] = kb;
  if (kb == P) {  // everything is selected
    for (int i = t; i < P; i += kThreads) out[i] = i;
    return;
  }
  const int forced_from = P - min(c.force_recent, kb);  // pages from here on are always selected
  const int groups = (P + kGroupPages - 1) / kGroupPages;

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
  if (kept_groups > kMaxGroups) {  // uniform; masses of equal scores: select by re-reading the row
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
    __syncthreads();  // wave_min and wave_max have been read by all
    if (lane == 0) { sh.wave_min[wave] = kmin; sh.wave_max[wave] = kmax; }
    constexpr int kBuckets = SelectShared<kThreads>::kBuckets;
    for (int i = t; i < kBuckets + kBuckets / 4; i += kThreads) sh.hist[i] = 0;
    if (t == 0) sh.ncand = 0;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) { kmin = min(kmin, sh.wave_min[w]); kmax = max(kmax, sh.wave_max[w]); }
    select_reread<kThreads>(key_of, P, kb, bucket_map(kmin, kmax, kBuckets), out, sh);
    return;
  }
#pragma unroll
  for (int v = 0; v < kGroupVecs; ++v) {
    int at = gplace[v];
#pragma unroll
    for (int i = 0; i < 4; ++i) at = lanes_before(__ballot(gkey[4 * v + i] >= T0), at);
#pragma unroll
    for (int i = 0; i < 4; ++i) {  // without branches: they cost more than the stores that they save
      const bool in = gkey[4 * v + i] >= T0;
      group_list[in ? at : kMaxGroups + lane] = group_of(4 * v + i);
      at += in;
    }
  }
  __syncthreads();

  // ---- 3. their scores: load (v, thread) is the half (thread % 2) of a group, so the pages ascend with (v, thread)
  uint32_t key[4 * kVecs];
  int first[kVecs];  // first page of the load
  const int loads = (2 * kept_groups + kThreads - 1) / kThreads;  // loads that any thread has
  {
    float4 raw[kVecs];
#pragma unroll
    for (int v = 0; v < kVecs; ++v) {
      const int at = (v * kThreads + t) / 2;
      first[v] = at < kept_groups ? group_list[at] * kGroupPages + (t % 2) * 4 : P;
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
  if (total > kKept) {  // uniform
    __syncthreads();    // the counts have been read by all
    select_spread<kThreads, kVecs, 4>(key, T0 - 1u, top, kb, [&](int at, int j) { out[at] = first[j / 4] + j % 4; }, counts[0], counts[1],
                                      turns);
    return;
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
      kept[in ? at : kKept + lane] = make_uint2(key[4 * v + i], (uint32_t)(first[v] + i));
      at += in;
    }
  }
  __syncthreads();

  // ---- 5. the k-th of them: one wave alone, whose rounds need no barrier, while they fit its registers
  // (stores at -1 lie outside the buffer and are dropped, which costs less than a branch)
  const __amdgpu_buffer_rsrc_t list = __builtin_amdgcn_make_buffer_rsrc(out, 0, kb * 4, 0x27000);
  auto emit = [&](int, int at, int page) { __builtin_amdgcn_raw_buffer_store_b32(page, list, at * 4, 0, 0); };
  if (total <= 24 * kWave) {
    if (wave > 0) return;
    if (total <= 4 * kWave) select_gathered<4>(kept, total, T0 - 1u, top, kb, emit);
    else if (total <= 8 * kWave) select_gathered<8>(kept, total, T0 - 1u, top, kb, emit);
    else if (total <= 16 * kWave) select_gathered<16>(kept, total, T0 - 1u, top, kb, emit);
    else select_gathered<24>(kept, total, T0 - 1u, top, kb, emit);
    return;
  }
  constexpr int kDense = kKept / kThreads;
  uint32_t dkey[kDense];
  int dpage[kDense];
#pragma unroll
  for (int j = 0; j < kDense; ++j) {
    const uint2 e = kept[j * kThreads + t];  // (what lies behind the last one is not used)
    dkey[j] = j * kThreads + t < total ? e.x : 0u;
    dpage[j] = (int)e.y;
  }
  select_spread<kThreads, kDense, 1>(dkey, T0 - 1u, top, kb, [&](int at, int j) { out[at] = dpage[j]; },
                                     counts[0], counts[1], turns);
}

}  // namespace

// Worth it while the kept groups are a small part of the row and fit the workgroup's registers (2048 of them, k and a quarter
// and some more). Kernel us of select.hip / this one, planted normal scores, 8 rows: 4097 pages, k 64 7.5 / 5.4; 8192, 64 8.6 / 5.4;
// 8192, 256 8.9 / 6.7; 12000, 500 12.0 / 9.4; 16384, 64 9.7 / 6.0; 32768, 64 13.9 / 6.9; 62501, 64 27.0 / 8.5; 62501, 1024 29.4 /
// 14.0; 125001, 1024 44.8 / 17.1; and 128 rows: 16384, 680 13.8 / 12.8. Not worth it: 4097, 340 7.6 / 7.7; 16384, 1024 (128 rows)
// 14.0 / 16.4; 62501, 2000 44.6 / 176 (too many groups). The maxima cost the score kernel 0.3 us (1 us of 90 at 16 x 16384 pages).
// Masses of equal scores that more groups reach are selected by re-reading: 16 x 62501 scores of five values 85 / 288.
bool select_uses_groups(const CacheView& c, int top_k) {
  const int P = c.max_pages_hint;
  return P > 4096 && P <= 131072 && top_k <= std::min(P / 24, 1280);
}

hipError_t launch_select_grouped(const CacheView& c, const float* d_scores, const uint32_t* d_group_max, int score_stride,
                                 int top_k, int32_t* d_sel_pages, int32_t* d_sel_count, hipStream_t stream) {
  const int P = c.max_pages_hint;
  auto go = [&](auto threads, auto vecs) {
    constexpr int kThreads = decltype(threads)::value, kVecs = decltype(vecs)::value;
    topk_select_grouped_kernel<kThreads, kVecs><<<dim3(c.B * c.Hkv), dim3(kThreads), 0, stream>>>(
        c, d_scores, d_group_max, score_stride, top_k, d_sel_pages, d_sel_count);
    return hipGetLastError();
  };
  const std::integral_constant<int, 512> wide;
  if (P <= 8192) return go(std::integral_constant<int, 256>(), std::integral_constant<int, 1>());
  if (P <= 16384) return go(wide, std::integral_constant<int, 1>());
  if (P <= 32768) return go(wide, std::integral_constant<int, 2>());
  if (P <= 65536) return go(wide, std::integral_constant<int, 4>());
  return go(wide, std::integral_constant<int, 8>());
}

}  // namespace unique
