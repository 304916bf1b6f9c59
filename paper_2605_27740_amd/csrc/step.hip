// Selection and attention of a decode step in one kernel: every workgroup of a row's chunks selects the row's top-k pages for
// itself (select_small.hpp) and attends over its chunk of them (decode_core.hpp); the first chunk's workgroup also writes the
// list out. A launch and the round trips between the two kernels fall away: the list stays in the LDS, the physical page
// beside each entry, looked up while the search for the k-th key runs. Of short rows every workgroup makes the scores, too.
// Scores, selection and attention are those of the separate kernels, in the same order: the same bits.
// What bounds it where the launch is small is a chain of latencies: the arguments, the length and the scores, the bound T0, the keys
// from it on, the k-th of them, the list, and one page per wave. Kernel us for one sequence of 2048 pages, k = 128: selection and
// attention apart 5.0 + 5.1, so 8.0.
#include "decode_core.hpp"
#include "score_core.hpp"
#include "select_groups.hpp"
#include "step_rule.hpp"

namespace unique {
namespace {

constexpr int kThreads = kDecWaves * kWave;

template <typename T, int D, int G, typename Select>
struct StepShared {
  Select sel;                       // apart from `dec`: a wave may be done before another one has its list
  DecodeShared<T, D, G> dec;
  int2 list[kStepMaxTopK + kWave];  // physical page, logical page; the last ones are for lanes without an entry
};

// What a step does to one chunk once the scores are known. select(kb, page_table, emit_all) selects kb < P pages: it calls emit_all in
// every wave for all that its lanes hold (see select_gathered). All threads call it.
template <typename T, int D, int S, int G, bool kNT, typename Shared, typename Select>
__device__ __forceinline__ void select_and_attend(const CacheView& c, const T* __restrict__ q, int split, int hkv, int b, int N, int P,
                                                  int top_k, int32_t* __restrict__ sel_pages, int32_t* __restrict__ sel_count,
                                                  const SplitPlan& plan, float scale_log2, const ChunkOut<T>& to, Shared& sh,
                                                  Select select) {
  const int row = b * c.Hkv + hkv;
  const int t = threadIdx.x, lane = t % kWave, wave = __builtin_amdgcn_readfirstlane(t / kWave);  // wave: scalar
  const int32_t* pt = c.page_table + (int64_t)b * c.max_pages;
  const int kb = min(top_k, P);
  const int begin = split * plan.pages_per_split, end = min(begin + plan.pages_per_split, kb);
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
    for (int p = begin + t; p < end; p += kThreads) sh.list[p - begin] = make_int2(pt[p], p);
    __syncthreads();
  } else {
    // Every wave knows the whole selection. It keeps the entries that it will attend over itself (see decode_chunk), so no
    // barrier is needed before it reads them back.
    auto emit_all = [&](int r, int at, int page, int ph) {
      const bool mine = at >= begin && at < end && (at - begin) % kDecWaves == wave;
      sh.list[mine ? at - begin : kStepMaxTopK + lane] = make_int2(ph, page);
      if (split == 0 && r % kDecWaves == wave && at >= 0) sel_row[at] = page;
    };
    select(kb, pt, emit_all);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }

  auto lookup = [&](int e, bool, int& ph, int& ntok) {
    const int2 entry = sh.list[e - begin];
    if (entry.x >= 0 && (int64_t)entry.x < c.num_phys) {
      ph = entry.x;
      ntok = min(S, N - entry.y * S);
    }
  };
  const Chunk chunk = {hkv, b, begin, end, N, (int64_t)row * plan.num_splits + split};
  decode_chunk<D, S, G, kNT>(c, q, chunk, wave, lane, lookup, scale_log2, to, sh.dec);
}

// The selection from scores in registers, row_page(j) for raw[j / 4].
template <int kVecs>
struct SelectFromScores {
  const CacheView& c;
  const float4 (&raw)[kVecs];
  int P;
  SmallShared<kThreads, kVecs>& sh;
  template <typename EmitAll>
  __device__ __forceinline__ void operator()(int kb, const int32_t* page_table, EmitAll emit_all) const {
    uint32_t key[4 * kVecs];
#pragma unroll
    for (int v = 0; v < kVecs; ++v) keys_of(raw[v], P - row_page<kThreads, 4>(4 * v), key + 4 * v);
    force_recent_keys<kThreads, kVecs, 4>(key, P, kb, c.force_recent);
    select_small<kThreads, kVecs>(key, P, kb, page_table, emit_all, sh);
  }
};

// Workgroups on a compute unit that the registers are held down for.
template <typename T, int D, int S>
constexpr int step_workgroups() { return step_held(sizeof(T) == 2, D, S) ? 3 : 1; }

// kVecs: 16-byte loads of scores per thread.
template <typename T, int D, int S, int G, bool kNT, int kVecs>
__global__ __launch_bounds__(kThreads, (step_workgroups<T, D, S>())) void select_decode_kernel(
    CacheView c, const T* __restrict__ q, const float* __restrict__ scores, int score_stride, int top_k,
    int32_t* __restrict__ sel_pages, int32_t* __restrict__ sel_count, SplitPlan plan, float scale_log2,
    float* __restrict__ part_o, float* __restrict__ part_ml, T* __restrict__ out, float* __restrict__ lse_out) {
  __shared__ StepShared<T, D, G, SmallShared<kThreads, kVecs>> sh;
  int split, hkv, b;
  locate_chunk(c, plan, split, hkv, b);
  // the scores are requested together with the sequence length: score rows are as long as the launch's bound on the pages
  const float* srow = scores + ((int64_t)b * c.Hkv + hkv) * score_stride;
  float4 raw[kVecs];
#pragma unroll
  for (int v = 0; v < kVecs; ++v) {
    const int p = row_page<kThreads, 4>(4 * v);
    raw[v] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (p < score_stride) raw[v] = *reinterpret_cast<const float4*>(srow + p);
  }
  const int N = c.seq_lens[b];
  const int P = min(min((N + S - 1) / S, c.max_pages_hint), kThreads * 4 * kVecs);
  const ChunkOut<T> to = {part_o, part_ml, out, lse_out, plan.num_splits};
  select_and_attend<T, D, S, G, kNT>(c, q, split, hkv, b, N, P, top_k, sel_pages, sel_count, plan, scale_log2, to, sh,
                                     SelectFromScores<kVecs>{c, raw, P, sh.sel});
}

// The same for longer rows, from the maxima of their groups of pages.
constexpr int kGroupVecs = kStepMaxGroupPages / (4 * kGroupPages * kThreads);
struct SelectFromGroups {
  const CacheView& c;
  const float* srow;
  const uint32_t* grow;
  int P;
  using Shared = GroupShared<kThreads, 4, kSmallCap>;
  static_assert(kStepMaxTopK <= kSmallCap && 9 * kStepMaxTopK <= 8 * Shared::kMaxGroups, "gather_from_groups");
  Shared& sh;
  template <typename EmitAll>
  __device__ __forceinline__ void operator()(int kb, const int32_t* page_table, EmitAll emit_all) const {
    const Gathered got = gather_from_groups<kThreads, kGroupVecs>(srow, grow, P, kb, P - min(c.force_recent, kb), sh);
    select_kept(sh.kept, got.total, got.T0 - 1u, kb, page_table, emit_all);
  }
};

template <typename T, int D, int S, int G, bool kNT>
__global__ __launch_bounds__(kThreads, (step_workgroups<T, D, S>())) void select_groups_decode_kernel(
    CacheView c, const T* __restrict__ q, const float* __restrict__ scores, const uint32_t* __restrict__ group_max, int score_stride,
    int top_k, int32_t* __restrict__ sel_pages, int32_t* __restrict__ sel_count, SplitPlan plan, float scale_log2,
    float* __restrict__ part_o, float* __restrict__ part_ml, T* __restrict__ out, float* __restrict__ lse_out) {
  __shared__ StepShared<T, D, G, SelectFromGroups::Shared> sh;
  int split, hkv, b;
  locate_chunk(c, plan, split, hkv, b);
  const int64_t row = (int64_t)b * c.Hkv + hkv;
  const int N = c.seq_lens[b];
  const int P = min(min((N + S - 1) / S, c.max_pages_hint), kStepMaxGroupPages);
  const ChunkOut<T> to = {part_o, part_ml, out, lse_out, plan.num_splits};
  select_and_attend<T, D, S, G, kNT>(
      c, q, split, hkv, b, N, P, top_k, sel_pages, sel_count, plan, scale_log2, to, sh,
      SelectFromGroups{c, scores + row * score_stride, group_max + row * (score_stride / kGroupPages), P, sh.sel});
}

// The whole step of a small launch in one kernel: every workgroup also scores its row's pages, with the arithmetic and in the
// lanes of the score kernel. The last page's statistics are refreshed by one wave, which scores that page with them; the first
// chunk's workgroup stores them (the others' loads of that record are not used).
template <typename T, typename TS, int D, int S, int G>
__global__ __launch_bounds__(kThreads) void whole_step_kernel(
    CacheView c, const T* __restrict__ q, float lambda, int refresh_tail, int top_k, int32_t* __restrict__ sel_pages,
    int32_t* __restrict__ sel_count, SplitPlan plan, float scale_log2, float* __restrict__ part_o, float* __restrict__ part_ml,
    T* __restrict__ out, float* __restrict__ lse_out) {
  using Scorer = RowScorer<T, TS, D, G>;
  constexpr int kChunks = Scorer::kChunks, kE = Scorer::kE;
  constexpr int kSteps = G == 8 ? 2 : 4;                     // rows in flight per lane (eight queries leave fewer registers)
  constexpr int kStepPages = kDecWaves * kRowsPerWave;       // pages that the workgroup scores at a time
  __shared__ StepShared<T, D, G, SmallShared<kThreads, 1>> sh;
  __shared__ __attribute__((aligned(16))) float row_scores[kStepWholePages];
  __shared__ __attribute__((aligned(16))) TS tail_mean[D];

  int split, hkv, b;
  locate_chunk(c, plan, split, hkv, b);
  const int t = threadIdx.x, lane = t % kWave, wave = __builtin_amdgcn_readfirstlane(t / kWave);  // wave: scalar
  const int row8 = lane / kRowLanes, cl = lane % kRowLanes;
  const int32_t* pt = c.page_table + (int64_t)b * c.max_pages;
  auto page_at = [&](int st) { return (st * kDecWaves + wave) * kRowsPerWave + row8; };
  int ids[kSteps];
  auto request_ids = [&](int st0) {
#pragma unroll
    for (int u = 0; u < kSteps; ++u) ids[u] = page_at(st0 + u) < c.max_pages_hint ? pt[page_at(st0 + u)] : -1;
  };
  request_ids(0);
  Scorer scorer;
  scorer.request(q + ((int64_t)b * c.H + hkv * G) * D, cl);
  const int N = c.seq_lens[b];
  const int P = min(min((N + S - 1) / S, c.max_pages_hint), kStepWholePages);

  // the last page: its keys are on their way while the other pages are scored
  constexpr int kTailWave = kDecWaves - 1;
  PageRefresh<T, D, S> tail;
  const int n_tail = min(S, N - (P - 1) * S);
  int tail_phys = -1;
  if (refresh_tail && wave == kTailWave && P > 0 && n_tail > 0) {  // uniform
    tail_phys = pt[P - 1];
    if (tail_phys < 0 || (int64_t)tail_phys >= c.num_phys) tail_phys = -1;
    else tail.request(reinterpret_cast<const T*>(c.k_cache) + (int64_t)tail_phys * c.kv_page_stride + (int64_t)hkv * c.kv_head_stride, n_tail, lane);
  }

  char* stats = reinterpret_cast<char*>(c.page_stats);
  const int64_t std_off = (int64_t)c.Hkv * D * (int64_t)sizeof(TS);  // byte offset of the stds inside a record
  const int steps = (P + kStepPages - 1) / kStepPages;
  bool first = true;
  for (int st0 = 0; st0 < steps; st0 += kSteps) {
    Raw16 md[kSteps][kChunks];
    float sd[kSteps];
    bool valid[kSteps];
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {  // a row without a page reads the first bytes of the statistics
      valid[u] = page_at(st0 + u) < P && ids[u] >= 0 && (int64_t)ids[u] < c.num_phys;
      const char* rec = stats + (valid[u] ? (int64_t)ids[u] : 0) * c.rec_bytes;
      const TS* src = reinterpret_cast<const TS*>(rec) + hkv * D + cl * kE;
#pragma unroll
      for (int j = 0; j < kChunks; ++j) md[u][j] = load_raw(src + j * (kE * kRowLanes));
      sd[u] = reinterpret_cast<const float*>(rec + std_off)[hkv];
    }
    request_ids(st0 + kSteps);
    if (first) scorer.unpack(lambda);
    first = false;
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
      const float s = scorer.score(md[u], sd[u]);
      const int p = page_at(st0 + u);
      const bool fresh = refresh_tail && p == P - 1 && valid[u] && n_tail > 0;  // the tail wave's
      // a page whose table entry points outside the pool gets NaN, which ranks below every score
      if (cl == 0 && p < P && !fresh) row_scores[p] = valid[u] ? s : __uint_as_float(0x7fc00000u);
    }
  }
  if (tail_phys >= 0) {  // uniform; the tail wave. (P > 0, so the queries have been unpacked.)
    tail.reduce(n_tail, lane);
    tail.store_mean(tail_mean, sizeof(TS) == 2, lane);
    if (split == 0) {
      char* rec = stats + (int64_t)tail_phys * c.rec_bytes;
      tail.store_mean(rec + (int64_t)hkv * D * (int)sizeof(TS), sizeof(TS) == 2, lane);
      if (lane == 0) reinterpret_cast<float*>(rec + std_off)[hkv] = tail.std;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    Raw16 md[kChunks];
#pragma unroll
    for (int j = 0; j < kChunks; ++j) md[j] = load_raw(&tail_mean[cl * kE + j * (kE * kRowLanes)]);
    const float s = scorer.score(md, tail.std);
    if (lane == 0) row_scores[P - 1] = s;
  }
  __syncthreads();
  const float4 raw[1] = {*reinterpret_cast<const float4*>(&row_scores[min(4 * t, kStepWholePages - 4)])};
  const ChunkOut<T> to = {part_o, part_ml, out, lse_out, plan.num_splits};
  select_and_attend<T, D, S, G, false>(c, q, split, hkv, b, N, P, top_k, sel_pages, sel_count, plan, scale_log2, to, sh,
                                       SelectFromScores<1>{c, raw, P, sh.sel});
}

template <typename T, int D, int S, int G>
hipError_t launch_t(const CacheView& c, const StepArgs& a, hipStream_t st) {
  const int rows = c.B * c.Hkv;
  const SplitPlan plan = selection_plan(c, a.top_k);
  const bool stream_nt = decode_streams(c, a.top_k);
  float* part_ml = a.partials + (size_t)rows * plan.num_splits * G * D;
  const int64_t list_bytes = (int64_t)std::min(a.top_k, c.max_pages_hint) * S * D * 2 * (int)sizeof(T);
  auto go = [&](auto kernel, size_t lds, auto... group_max) {
    const int extra = step_extra_lds(step_held(sizeof(T) == 2, D, S), plan.num_splits, list_bytes, (int)lds);
    const dim3 grid = plan.rotate ? dim3(c.Hkv, c.B, plan.num_splits) : dim3(plan.num_splits, c.Hkv, c.B);
    kernel<<<grid, dim3(kThreads), extra, st>>>(c, reinterpret_cast<const T*>(a.q), a.scores, group_max..., a.score_stride, a.top_k,
                                            a.sel_pages, a.sel_count, plan, decode_scale_log2(c, a.sm_scale), a.partials, part_ml,
                                            reinterpret_cast<T*>(a.out), a.lse_out);
    return hipGetLastError();
  };
  // rows that no kernel here is made for would be cut without a word
  if (a.top_k > kStepMaxTopK || c.max_pages_hint > (a.group_max ? kStepMaxGroupPages : kStepMaxPages)) return hipErrorInvalidValue;
  // A step, us, as it is / with plain loads of K and V where a launch streams: 60 x 1000 pages, k = 64 87.7 / 92.9, 12 x 3126, 200, G = 8
  // 71.9 / 76.3, 16 x 8192, 256 141.5 / 145.1, fp32 8 x 2000, 128 44.3 / 49.6; / with 16 scores per thread for all rows: 1 x 1000, 64
  // 17.2 / 18.9, 8 x 1024 23.3 / 24.4, 8 x 2048 30.0 / 30.8.
  if (a.group_max) {
    constexpr size_t kLds = sizeof(StepShared<T, D, G, SelectFromGroups::Shared>);
    return stream_nt ? go(select_groups_decode_kernel<T, D, S, G, true>, kLds, a.group_max)
                     : go(select_groups_decode_kernel<T, D, S, G, false>, kLds, a.group_max);
  }
  auto go_vecs = [&](auto vecs) {
    constexpr int kVecs = decltype(vecs)::value;
    constexpr size_t kLds = sizeof(StepShared<T, D, G, SmallShared<kThreads, kVecs>>);
    return stream_nt ? go(select_decode_kernel<T, D, S, G, true, kVecs>, kLds) : go(select_decode_kernel<T, D, S, G, false, kVecs>, kLds);
  };
  if (c.max_pages_hint <= 4 * kThreads) return go_vecs(std::integral_constant<int, 1>());
  if (c.max_pages_hint <= 8 * kThreads) return go_vecs(std::integral_constant<int, 2>());
  return go_vecs(std::integral_constant<int, 4>());
}

template <typename T, int D, int S, int G>
hipError_t launch_whole_t(const CacheView& c, const StepArgs& a, hipStream_t st) {
  if (a.top_k > kStepMaxTopK || c.max_pages_hint > kStepWholePages) return hipErrorInvalidValue;
  const SplitPlan plan = selection_plan(c, a.top_k);
  float* part_ml = a.partials + (size_t)c.B * c.Hkv * plan.num_splits * G * D;
  auto go = [&](auto kernel) {
    const dim3 grid = plan.rotate ? dim3(c.Hkv, c.B, plan.num_splits) : dim3(plan.num_splits, c.Hkv, c.B);
    kernel<<<grid, dim3(kThreads), 0, st>>>(c, reinterpret_cast<const T*>(a.q), a.lambda, a.refresh_tail, a.top_k, a.sel_pages,
                                            a.sel_count, plan, decode_scale_log2(c, a.sm_scale), a.partials, part_ml,
                                            reinterpret_cast<T*>(a.out), a.lse_out);
    return hipGetLastError();
  };
  return c.stats_bf16 ? go(whole_step_kernel<T, bf16_t, D, S, G>) : go(whole_step_kernel<T, float, D, S, G>);
}

template <typename T, int D, int S>
hipError_t dispatch_g(const CacheView& c, const StepArgs& a, hipStream_t st) {
  auto go = [&](auto group) {
    constexpr int G = decltype(group)::value;
    return a.scores ? launch_t<T, D, S, G>(c, a, st) : launch_whole_t<T, D, S, G>(c, a, st);
  };
  switch (c.H / c.Hkv) {
    case 1: return go(std::integral_constant<int, 1>());
    case 2: return go(std::integral_constant<int, 2>());
    case 4: return go(std::integral_constant<int, 4>());
    case 8: return go(std::integral_constant<int, 8>());
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// One translation unit per element type, head dimension and page size: UNIQUE_ELEM, UNIQUE_DIM, UNIQUE_PAGE.
template <>
hipError_t launch_select_decode<UNIQUE_ELEM, UNIQUE_DIM, UNIQUE_PAGE>(const CacheView& c, const StepArgs& a, hipStream_t st) {
  return dispatch_g<UNIQUE_ELEM, UNIQUE_DIM, UNIQUE_PAGE>(c, a, st);
}

}  // namespace unique
