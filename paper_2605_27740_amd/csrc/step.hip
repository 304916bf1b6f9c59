// Selection and attention of a decode step in one kernel: every workgroup of a row's chunks selects the row's top-k pages for
// itself (select_small.hpp) and attends over its chunk of them (decode_core.hpp); the first chunk's workgroup also writes the
// list out. A launch and the round trips between the two kernels fall away: the list stays in the LDS, the physical page
// beside each entry, looked up while the search for the k-th key runs.
// The selection is exact and the attention that of the decode kernel, in the same order: the same bits as in separate kernels.
// What bounds it where the launch is small is a chain of latencies: of 17 200 cycles of a workgroup for one sequence of 2048
// pages, k = 128, the arguments, length and scores take 1800, the keys 900, the bound T0 2100, gathering 1700, the k-th key
// 2200, the list 1600, the attention over one page per wave 6900. Kernel us, selection + attention apart 5.2 + 5.8, so 8.5.
#include "decode_core.hpp"
#include "select_small.hpp"
#include "step_rule.hpp"

namespace unique {
namespace {

constexpr int kThreads = kDecWaves * kWave;

// kVecs: 16-byte loads of scores per thread.
template <typename T, int D, int S, int G, bool kNT, int kVecs>
__global__ __launch_bounds__(kThreads) void select_decode_kernel(
    CacheView c, const T* __restrict__ q, const float* __restrict__ scores, int score_stride, int top_k,
    int32_t* __restrict__ sel_pages, int32_t* __restrict__ sel_count, SplitPlan plan, float scale_log2,
    float* __restrict__ part_o, float* __restrict__ part_ml, T* __restrict__ out, float* __restrict__ lse_out) {
  constexpr int kPer = 4, kItems = kVecs * kPer;
  __shared__ SmallShared<kThreads, kVecs> sel;  // apart from `dec`: a wave may be done before another one has its list
  __shared__ DecodeShared<T, D, G> dec;
  __shared__ int2 list[kStepMaxTopK + kWave];  // physical page, logical page; the last ones are for lanes without an entry

  int split, hkv, b;
  locate_chunk(c, plan, split, hkv, b);
  const int row = b * c.Hkv + hkv;
  const int t = threadIdx.x, lane = t % kWave, wave = __builtin_amdgcn_readfirstlane(t / kWave);  // wave: scalar
  // the scores are requested together with the sequence length: score rows are as long as the launch's bound on the pages
  auto page_of = [](int j) { return row_page<kThreads, kPer>(j); };
  const float* srow = scores + (int64_t)row * score_stride;
  const int32_t* pt = c.page_table + (int64_t)b * c.max_pages;
  float4 raw[kVecs];
#pragma unroll
  for (int v = 0; v < kVecs; ++v) {
    raw[v] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (page_of(4 * v) < score_stride) raw[v] = *reinterpret_cast<const float4*>(srow + page_of(4 * v));
  }
  const int N = c.seq_lens[b];
  const int P = min(min((N + S - 1) / S, c.max_pages_hint), kThreads * kItems);
  const int kb = min(top_k, P);
  const int begin = split * plan.pages_per_split, end = min(begin + plan.pages_per_split, kb);
  const ChunkOut<T> to = {part_o, part_ml, out, lse_out, plan.num_splits};
  int32_t* sel_row = sel_pages + (int64_t)row * top_k;
  if (split == 0) {
    for (int i = kb + t; i < top_k; i += kThreads) sel_row[i] = -1;
    if (t == 0) sel_count[row] = kb;
  }
  if (begin >= kb) {
    write_empty<T, D, G>(c, to, b, hkv);
    return;
  }

  if (kb == P) {  // every page is selected
    for (int p = t; p < P; p += kThreads)
      if (split == 0) sel_row[p] = p;
    for (int p = begin + t; p < end; p += kThreads) list[p - begin] = make_int2(pt[p], p);
    __syncthreads();
  } else {
    uint32_t key[kItems];
#pragma unroll
    for (int v = 0; v < kVecs; ++v) keys_of(raw[v], P - page_of(4 * v), key + 4 * v);
    force_recent_keys<kThreads, kVecs, kPer>(key, P, kb, c.force_recent);
    // Every wave knows the whole selection. It keeps the entries that it will attend over itself (see decode_chunk), so no
    // barrier is needed before it reads them back.
    auto emit_all = [&](int r, int at, int page, int ph) {
      const bool mine = at >= begin && at < end && (at - begin) % kDecWaves == wave;
      list[mine ? at - begin : kStepMaxTopK + lane] = make_int2(ph, page);
      if (split == 0 && r % kDecWaves == wave && at >= 0) sel_row[at] = page;
    };
    auto emit_own = [&](int at, int page) {
      if (split == 0) sel_row[at] = page;
      if (at >= begin && at < end) list[at - begin] = make_int2(pt[page], page);
    };
    select_small<kThreads, kVecs>(key, P, kb, pt, emit_all, emit_own, sel);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }

  auto lookup = [&](int e, bool, int& ph, int& ntok) {
    const int2 entry = list[e - begin];
    if (entry.x >= 0 && (int64_t)entry.x < c.num_phys) {
      ph = entry.x;
      ntok = min(S, N - entry.y * S);
    }
  };
  const Chunk chunk = {hkv, b, begin, end, N, (int64_t)row * plan.num_splits + split};
  decode_chunk<D, S, G, kNT>(c, q, chunk, wave, lane, lookup, scale_log2, to, dec);
}

template <typename T, int D, int S, int G>
hipError_t launch_t(const CacheView& c, const StepArgs& a, hipStream_t st) {
  const int rows = c.B * c.Hkv;
  const SplitPlan plan = selection_plan(c, a.top_k);
  const bool stream_nt = decode_streams(c, a.top_k);
  float* part_ml = a.partials + (size_t)rows * plan.num_splits * G * D;
  auto go = [&](auto kernel) {
    const dim3 grid = plan.rotate ? dim3(c.Hkv, c.B, plan.num_splits) : dim3(plan.num_splits, c.Hkv, c.B);
    kernel<<<grid, dim3(kThreads), 0, st>>>(c, reinterpret_cast<const T*>(a.q), a.scores, a.score_stride, a.top_k,
                                            a.sel_pages, a.sel_count, plan, decode_scale_log2(c, a.sm_scale), a.partials, part_ml,
                                            reinterpret_cast<T*>(a.out), a.lse_out);
    return hipGetLastError();
  };
  if (c.max_pages_hint <= 4 * kThreads)
    return stream_nt ? go(select_decode_kernel<T, D, S, G, true, 1>) : go(select_decode_kernel<T, D, S, G, false, 1>);
  if (c.max_pages_hint <= 8 * kThreads)
    return stream_nt ? go(select_decode_kernel<T, D, S, G, true, 2>) : go(select_decode_kernel<T, D, S, G, false, 2>);
  return stream_nt ? go(select_decode_kernel<T, D, S, G, true, 4>) : go(select_decode_kernel<T, D, S, G, false, 4>);
}

template <typename T, int D, int S>
hipError_t dispatch_g(const CacheView& c, const StepArgs& a, hipStream_t st) {
  switch (c.H / c.Hkv) {
    case 1: return launch_t<T, D, S, 1>(c, a, st);
    case 2: return launch_t<T, D, S, 2>(c, a, st);
    case 4: return launch_t<T, D, S, 4>(c, a, st);
    case 8: return launch_t<T, D, S, 8>(c, a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// One translation unit per element type and head dimension: UNIQUE_ELEM, UNIQUE_DIM.
template <>
hipError_t launch_select_decode<UNIQUE_ELEM, UNIQUE_DIM>(const CacheView& c, const StepArgs& a, hipStream_t st) {
  switch (c.S) {
    case 8: return dispatch_g<UNIQUE_ELEM, UNIQUE_DIM, 8>(c, a, st);
    case 16: return dispatch_g<UNIQUE_ELEM, UNIQUE_DIM, 16>(c, a, st);
    case 32: return dispatch_g<UNIQUE_ELEM, UNIQUE_DIM, 32>(c, a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace unique
