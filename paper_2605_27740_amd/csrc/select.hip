// Top-k page selection per (sequence, KV head) row (Section 3.2 of the paper, radix-based top-k).
//
// One workgroup per row; the row's scores are read once and stay in registers as order-preserving 32-bit keys (rows of
// more than 32768 pages are read twice or more, except up to 65536 pages with k > 1024). The paper narrows the k-th
// largest score with two 8-bit radix rounds over bf16 scores; here the scores are fp32 and the selected set has to equal
// an exact ranking. What bounds the kernel is a chain of latencies on one compute unit and, for long rows, the
// instructions spent per key (about 130 wave instructions per 64 keys if every key goes through every step), so the
// search is:
//   1. the row's extremes and a lower bound T0 of the k-th key: the smallest of the maxima of disjoint groups of keys,
//      of which there are at least k. 10 to 35 % of the keys are not below it. Where a thread holds 32 keys and
//      k is at most 1024 those are gathered in LDS and dealt out again, so the remaining steps see a few keys per thread.
//   2. one histogram pass over buckets that are LINEAR in the score between T0 and the row's maximum (a monotone map,
//      so bucket order never contradicts score order). It finds the bucket holding the k-th largest score; everything in
//      higher buckets is selected. Linear buckets spread page scores far better than the leading bits of a float (which
//      are mostly exponent), so LDS atomics see little same-address contention and the boundary bucket holds only a
//      handful of candidates. Every wave scans the histogram for itself, which saves two barriers.
//   3. exact resolution among the candidates of the boundary bucket: by ranking on (key, page index) when they are few
//      (up to 64: one per lane, every wave for itself; up to 512 or the workgroup's threads: one per thread, pairwise),
//      otherwise by four 8-bit radix rounds over their keys (this also covers degenerate rows such as all scores equal).
//   4. an index-ordered compaction that emits the selected logical pages in ascending order and takes keys tied with
//      the k-th from the lowest page index upward.
// Kernel us before (a thread owned consecutive pages, every key went through every step) and now, planted normal scores:
// 8 rows x 256 pages, k 16: 3.8 / 3.8; 8 x 2048, 128: 5.1 / 4.9; 128 x 8192, 256: 9.0 / 8.4; 640 x 4096, 64: 17.0 / 9.6;
// 16 x 16384, 1024: 13.5 / 12.7; 8 x 32768, 512: 22.4 / 15.0; 128 x 24000, 3000: 25.7 / 21.8; 8 x 62501, 1024: 67.8 / 29.7;
// 4 x 131072, 1024: 217 / 43; all scores equal, 128 x 8192: 44 / 20. A few sizes are slower: 8 x 4097, 16 7.2 / 7.6; 8 x 8193,
// 300 10.5 / 11.3; rows of 2600 pages under a bound of 131072 8.4 / 9.9; scores of five values, 16 x 131072 432 / 447.
#include <type_traits>

#include "select_core.hpp"

namespace unique {
namespace {

// One workgroup per row. kCompact: the keys that are not below T0 are gathered and dealt out again.
template <int kThreads, int kVecs, int kPer, bool kCompact>
__global__ __launch_bounds__(kThreads) void topk_select_kernel(CacheView c, const float* __restrict__ scores,
                                                               int score_stride, int top_k,
                                                               int32_t* __restrict__ sel_pages,
                                                               int32_t* __restrict__ sel_count) {
  using Sh = SelectShared<kThreads>;
  constexpr int kWaves = Sh::kWaves, kItems = kPer * kVecs;
  constexpr int kDense = 8;  // keys per thread that are kept when the others are dropped
  static_assert(kPer == 4 || (kPer == 1 && !kCompact), "scores per load");
  __shared__ Sh sh;
  __shared__ uint2 kept[kCompact ? kDense * kThreads : 1];

  const int row = blockIdx.x;
  const int b = row / c.Hkv;
  const int N = c.seq_lens[b];
  int P = min((N + c.S - 1) / c.S, c.max_pages_hint);
  P = min(P, kThreads * kItems);  // a row longer than the host bound is cut, never overrun
  const int kb = min(top_k, P);
  const int t = threadIdx.x, lane = t % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
  int32_t* out = sel_pages + (int64_t)row * top_k;
  const float* srow = scores + (int64_t)row * score_stride;

  for (int i = kb + t; i < top_k; i += kThreads) out[i] = -1;
  if (t == 0) sel_count[row] = kb;
  if (kb == P) {  // everything is selected
    for (int i = t; i < P; i += kThreads) out[i] = i;
    return;
  }

  auto page_of = [](int j) { return row_page<kThreads, kPer>(j); };
  uint32_t key[kItems];
  if constexpr (kPer == 1) {
    float raw[kVecs];
#pragma unroll
    for (int v = 0; v < kVecs; ++v) raw[v] = page_of(v) < P ? srow[page_of(v)] : 0.f;
#pragma unroll
    for (int v = 0; v < kVecs; ++v) key[v] = page_of(v) < P ? score_key(raw[v]) : 0u;
  } else {
    float4 raw[kVecs];
#pragma unroll
    for (int v = 0; v < kVecs; ++v) {
      const int p = page_of(4 * v);
      raw[v] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (p < P) raw[v] = *reinterpret_cast<const float4*>(srow + p);  // the row is padded to a multiple of 4
    }
#pragma unroll
    for (int v = 0; v < kVecs; ++v) keys_of(raw[v], P - page_of(4 * v), key + 4 * v);
  }
  force_recent_keys<kThreads, kVecs, kPer>(key, P, kb, c.force_recent);
  BucketMap map;
  const uint32_t T0 = bound_row<kThreads, kVecs, kPer>(key, P, kb, map, sh);

  if constexpr (kCompact) {
    // many keys per thread: the few that are not below T0 are gathered, in page order, and dealt out again
    int place[kVecs];
#pragma unroll
    for (int v = 0; v < kVecs; ++v) {
      int n = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) n += __popcll(__ballot(key[4 * v + i] >= T0));
      if (lane == 0) sh.sure_cnt[v * kWaves + wave] = n;
    }
    __syncthreads();
    const int total = wave_prefixes<kVecs, kWaves>(sh.sure_cnt, wave, place);
    if (total <= kDense * kThreads) {  // uniform
#pragma unroll
      for (int v = 0; v < kVecs; ++v) {
        int at = place[v];
#pragma unroll
        for (int i = 0; i < 4; ++i) at = lanes_before(__ballot(key[4 * v + i] >= T0), at);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (key[4 * v + i] >= T0) kept[at++] = make_uint2(key[4 * v + i], (uint32_t)page_of(4 * v + i));
      }
      __syncthreads();
      uint32_t dkey[kDense];
      int dpage[kDense];
#pragma unroll
      for (int j = 0; j < kDense; ++j) {
        const int at = j * kThreads + t;
        const uint2 e = at < total ? kept[at] : make_uint2(0u, 0x7fffffffu);
        dkey[j] = e.x;
        dpage[j] = (int)e.y;
      }
      select_keys<kThreads, kDense, 1>(dkey, [&](int j) { return dpage[j]; }, T0, map, kb,
                                       [&](int at, int j) { out[at] = dpage[j]; }, sh);
      return;
    }
  }
  select_keys<kThreads, kVecs, kPer>(key, page_of, T0, map, kb, [&](int at, int j) { out[at] = page_of(j); }, sh);
}

// Rows of more keys than the registers hold: the row is read twice in chunks of 32 keys per thread, once for the bound
// T0 and the extremes and once to gather the keys that are not below T0 in the LDS, in page order; the selection then
// runs on those. Rows that leave too many (more than kDense * kThreads: a very large k, or masses of equal scores) are
// selected by re-reading.
template <int kThreads>
__global__ __launch_bounds__(kThreads) void topk_select_long_kernel(CacheView c, const float* __restrict__ scores,
                                                                    int score_stride, int top_k,
                                                                    int32_t* __restrict__ sel_pages,
                                                                    int32_t* __restrict__ sel_count) {
  using Sh = SelectShared<kThreads>;
  constexpr int kWaves = Sh::kWaves, kBuckets = Sh::kBuckets;
  constexpr int kVecs = 8, kUnitVecs = 4;      // 16-byte loads per thread and chunk; units of the groups for T0
  constexpr int kChunk = kVecs * 4 * kThreads, kUnit = kUnitVecs * 4 * kThreads;
  constexpr int kDense = 16;
  __shared__ Sh sh;
  __shared__ uint2 kept[kDense * kThreads];

  const int row = blockIdx.x;
  const int b = row / c.Hkv;
  const int N = c.seq_lens[b];
  const int P = min((N + c.S - 1) / c.S, c.max_pages_hint);
  const int kb = min(top_k, P);
  const int t = threadIdx.x, lane = t % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
  int32_t* out = sel_pages + (int64_t)row * top_k;
  const float* srow = scores + (int64_t)row * score_stride;

  for (int i = kb + t; i < top_k; i += kThreads) out[i] = -1;
  if (t == 0) sel_count[row] = kb;
  if (kb == P) {
    for (int i = t; i < P; i += kThreads) out[i] = i;
    return;
  }
  const int forced_from = P - min(c.force_recent, kb);  // pages from here on are always selected

  uint32_t key[4 * kVecs];
  auto page_of = [&](int chunk, int j) { return chunk * kChunk + (j / 4) * 4 * kThreads + 4 * t + j % 4; };
  auto load_chunk = [&](int chunk) {  // keys of the chunk; 0 past the row's end
    float4 raw[kVecs];
#pragma unroll
    for (int v = 0; v < kVecs; ++v) {
      const int p = page_of(chunk, 4 * v);
      raw[v] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (p < P) raw[v] = *reinterpret_cast<const float4*>(srow + p);  // the row is padded to a multiple of 4
    }
#pragma unroll
    for (int v = 0; v < kVecs; ++v) keys_of(raw[v], P - page_of(chunk, 4 * v), key + 4 * v);
    if ((chunk + 1) * kChunk > forced_from) {
#pragma unroll
      for (int j = 0; j < 4 * kVecs; ++j)
        if (page_of(chunk, j) >= forced_from && page_of(chunk, j) < P) key[j] = kKeyForced;
    }
  };
  const int chunks = (P + kChunk - 1) / kChunk;

  // Groups for T0 (see the register kernel): a thread's keys in `per_group` consecutive units, `groups` of them per
  // thread, the last one with all that follows; with one group per thread, those of 2^n threads together.
  const int units = P / kUnit, groups = units * kThreads >= kb ? (kb + kThreads - 1) / kThreads : 0;
  const int per_group = groups > 0 ? units / groups : 0;
  uint32_t kmin = 0xffffffffu, kmax = 0u, low = 0xffffffffu, group_max = 0u;
  auto key_of = [&](int page) { return page >= forced_from ? kKeyForced : score_key(srow[page]); };
  if (units == 0) {  // a short row of a long launch, which will be re-read: the extremes alone (2600 pages: 12.9 -> 10.1 us)
    for (int p0 = 0; p0 < P; p0 += 8 * kThreads) {
      uint32_t kk[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) kk[u] = p0 + u * kThreads + t < P ? key_of(p0 + u * kThreads + t) : 0u;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (p0 + u * kThreads >= P) break;  // uniform
        const bool finite = kk[u] > kKeyNegInf && kk[u] < kKeyPosInf;
        kmin = min(kmin, finite ? kk[u] : 0xffffffffu);
        kmax = max(kmax, finite ? kk[u] : 0u);
      }
    }
  }
  for (int ch = 0; ch < chunks && units > 0; ++ch) {
    load_chunk(ch);
#pragma unroll
    for (int u = 0; u < kVecs / kUnitVecs; ++u) {
      const int unit = ch * (kVecs / kUnitVecs) + u;
      if (unit > 0 && per_group > 0 && unit % per_group == 0 && unit / per_group < groups) {
        low = min(low, group_max);
        group_max = 0u;
      }
#pragma unroll
      for (int i = 0; i < 4 * kUnitVecs; ++i) {
        const uint32_t k = key[u * 4 * kUnitVecs + i];
        const bool finite = k > kKeyNegInf && k < kKeyPosInf;
        kmin = min(kmin, finite ? k : 0xffffffffu);
        kmax = max(kmax, finite ? k : 0u);
        group_max = max(group_max, k);
      }
    }
  }
  {
    auto merge = [&](int lanes, uint32_t other) { if (lanes * kb <= kThreads) group_max = max(group_max, other); };
    merge(2, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)group_max, kDppXor1, 0xf, 0xf, true));
    merge(4, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)group_max, kDppXor2, 0xf, 0xf, true));
    merge(8, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)group_max, kDppHalfMirror, 0xf, 0xf, true));
    merge(16, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)group_max, kDppMirror, 0xf, 0xf, true));
    low = groups > 0 ? min(low, group_max) : 0u;
  }
  kmin = wave_allreduce_minmax<false>(kmin);
  kmax = wave_allreduce_minmax<true>(kmax);
  low = wave_allreduce_minmax<false>(low);
  if (lane == 0) { sh.wave_min[wave] = kmin; sh.wave_max[wave] = kmax; sh.wave_low[wave] = low; }
  for (int i = t; i < kBuckets + kBuckets / 4; i += kThreads) sh.hist[i] = 0;
  if (t == 0) sh.ncand = 0;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    kmin = min(kmin, sh.wave_min[w]); kmax = max(kmax, sh.wave_max[w]); low = min(low, sh.wave_low[w]);
  }
  const uint32_t T0 = max(low, 1u);

  int total = groups > 0 ? 0 : kDense * kThreads + 1;  // keys kept so far
  for (int ch = 0; ch < chunks && total <= kDense * kThreads; ++ch) {  // uniform
    load_chunk(ch);
    int* counts = ch % 2 ? sh.tie_cnt : sh.sure_cnt;  // alternating, so one barrier per chunk is enough
#pragma unroll
    for (int v = 0; v < kVecs; ++v) {
      int n = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) n += __popcll(__ballot(key[4 * v + i] >= T0));
      if (lane == 0) counts[v * kWaves + wave] = n;
    }
    __syncthreads();
    int place[kVecs];
    const int here = wave_prefixes<kVecs, kWaves>(counts, wave, place);
    if (total + here <= kDense * kThreads) {
#pragma unroll
      for (int v = 0; v < kVecs; ++v) {
        int at = total + place[v];
#pragma unroll
        for (int i = 0; i < 4; ++i) at = lanes_before(__ballot(key[4 * v + i] >= T0), at);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (key[4 * v + i] >= T0) kept[at++] = make_uint2(key[4 * v + i], (uint32_t)page_of(ch, 4 * v + i));
      }
    }
    total += here;
  }
  __syncthreads();
  if (total > kDense * kThreads) {
    select_reread<kThreads>(key_of, P, kb, bucket_map(kmin, kmax, kBuckets), [&](int at, int page) { out[at] = page; }, sh);
    return;
  }
  uint32_t dkey[kDense];
  int dpage[kDense];
#pragma unroll
  for (int j = 0; j < kDense; ++j) {
    const int at = j * kThreads + t;
    const uint2 e = at < total ? kept[at] : make_uint2(0u, 0x7fffffffu);
    dkey[j] = e.x;
    dpage[j] = (int)e.y;
  }
  if (T0 > kKeyNegInf && T0 < kKeyPosInf) kmin = T0;
  select_keys<kThreads, kDense, 1>(dkey, [&](int j) { return dpage[j]; }, T0, bucket_map(kmin, kmax, kBuckets), kb,
                                   [&](int at, int j) { out[at] = dpage[j]; }, sh);
}

template <int kN>
using Int = std::integral_constant<int, kN>;

// Gathering by default where a thread holds 32 keys: fewer gain nothing, 64 leave no registers for the second set.
template <int kThreads, int kVecs, int kPer = 4, bool kCompact = kVecs * kPer == 32>
hipError_t launch_t(const CacheView& c, const float* scores, int stride, int top_k, int32_t* sel, int32_t* cnt,
                    hipStream_t st) {
  topk_select_kernel<kThreads, kVecs, kPer, kCompact><<<dim3(c.B * c.Hkv), dim3(kThreads), 0, st>>>(
      c, scores, stride, top_k, sel, cnt);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_select(const CacheView& c, const float* d_scores, const uint32_t* d_group_max, int score_stride, int top_k,
                         int32_t* d_sel_pages, int32_t* d_sel_count, hipStream_t stream) {
  if (d_group_max)
    return launch_select_grouped(c, d_scores, d_group_max, score_stride, top_k, d_sel_pages, d_sel_count, stream);
  const int P = c.max_pages_hint;
  auto go = [&](auto threads, auto vecs) {
    return launch_t<decltype(threads)::value, decltype(vecs)::value>(c, d_scores, score_stride, top_k, d_sel_pages,
                                                                     d_sel_count, stream);
  };
  const int rows = c.B * c.Hkv;
  // The smallest workgroup whose registers hold the row, unless another one measured faster; kernel us on rows of
  // planted normal scores (rows x pages, k):
  //   8 x 256, 16: 3.8 with 256 threads and one key each, 4.1 with one wave; 640 x 256, 4: 4.6 and 4.3
  //   640 x 4096, 64: 9.5 with 512 threads, 19 with 1024 (two workgroups of 1024 per compute unit: a second round)
  //   8 x 2048, 128: 5.4 with 256 threads, 4.9 with 512; 512 x 2048, 64: 7.0 and 7.6
  //   128 x 8192, 256: 8.4 with 512 threads, 9.2 with 1024; with k = 1024 10.8 and 10.0, but at 512 rows 14.2 and 18.5 and
  //   at 8 x 4097 8.4 and 8.9 (8 x 6000: 9.2 and 9.0)
  //   16 x 16384, 256: 10.3 with 512 threads, 11.7 with 1024; with k = 512 17 and 12.2, as a group for T0 is then a
  //   single thread's keys and more of them are left; 640 x 8193, 512: 20.8 and 32.5, two rounds again
  //   16 x 32768 and k above the 1024 threads, without a bound: 25.7 with a vain attempt to gather, 20.6 without
  if (P <= 256 && rows <= 512) return launch_t<256, 1, 1>(c, d_scores, score_stride, top_k, d_sel_pages, d_sel_count, stream);
  if (P <= 256) return go(Int<64>(), Int<1>());
  if (P <= 1024) return go(Int<256>(), Int<1>());
  if (P <= 2048) return rows > 256 ? go(Int<256>(), Int<2>()) : go(Int<512>(), Int<1>());
  if (P <= 4096) return go(Int<512>(), Int<2>());
  if (P <= 8192) return rows <= 256 && top_k > 512 && P > 5120 ? go(Int<1024>(), Int<2>()) : go(Int<512>(), Int<4>());
  if (P <= 16384) return top_k <= (rows > 256 ? 512 : 256) ? go(Int<512>(), Int<8>()) : go(Int<1024>(), Int<4>());
  if (P <= 32768 && top_k > 1024)
    return launch_t<1024, 8, 4, false>(c, d_scores, score_stride, top_k, d_sel_pages, d_sel_count, stream);
  if (P <= 32768) return go(Int<1024>(), Int<8>());
  // Beyond that the long kernel (8 x 62501, 1024: 30 us; 48 with all keys in registers), but it re-reads rows that leave
  // too many keys above T0, which at these lengths is the rule from about k = 2000 on (8 x 65536, 2048: 117 us against 48)
  if (P <= 65536 && top_k > 1024) return go(Int<1024>(), Int<16>());
  topk_select_long_kernel<1024><<<dim3(c.B * c.Hkv), dim3(1024), 0, stream>>>(c, d_scores, score_stride, top_k,
                                                                              d_sel_pages, d_sel_count);
  return hipGetLastError();
}

}  // namespace unique
