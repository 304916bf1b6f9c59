// Top-k selection for long rows whose group maxima the score kernel has left beside the scores (one key per 8 pages).
//
// A row belongs to one workgroup, whose loads bound the selection of a long row: 62501 scores are 250 KB for one compute unit,
// read twice. Here the maxima are read instead. At least k groups reach the k-th largest of them, T0, so the k-th score does,
// too, and only the groups that reach T0 -- about k -- can hold a selected page: their scores alone are read, an eighth of the row
// plus 8 k of them. T0 and then the exact k-th key are found by bisection over keys in registers. One wave makes the last step,
// whose rounds would need barriers of all the others. What bounds it is that chain of steps on one compute unit.
#include <algorithm>
#include <type_traits>

#include "select_groups.hpp"
#include "step_rule.hpp"

namespace unique {
namespace {

// kGroupVecs: 16-byte loads of group maxima per thread.
template <int kThreads, int kGroupVecs>
__global__ __launch_bounds__(kThreads) void topk_select_grouped_kernel(CacheView c, const float* __restrict__ scores,
                                                                       const uint32_t* __restrict__ group_max,
                                                                       int score_stride, int top_k,
                                                                       int32_t* __restrict__ sel_pages,
                                                                       int32_t* __restrict__ sel_count) {
  constexpr int kVecs = 8;            // 16-byte loads of scores per thread
  constexpr int kKept = 24 * kWave;   // keys from T0 on: what one wave holds
  __shared__ GroupShared<kThreads, kVecs, kKept> sh;
  // the largest k of such rows fits (see gather_from_groups)
  constexpr int kMostPages = kThreads * kGroupVecs * 4 * kGroupPages;
  constexpr int kMostK = kMostPages / kGroupsPagesPerK < kGroupsMaxTopK ? kMostPages / kGroupsPagesPerK : kGroupsMaxTopK;
  static_assert(kMostK <= kKept && 9 * kMostK <= 8 * GroupShared<kThreads, kVecs, kKept>::kMaxGroups, "");

  const int row = blockIdx.x;
  const int b = row / c.Hkv;
  const int t = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const int N = c.seq_lens[b];
  int P = min((N + c.S - 1) / c.S, c.max_pages_hint);
  P = min(P, kMostPages);  // a row longer than the host bound is cut, never overrun
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
  const Gathered got = gather_from_groups<kThreads, kGroupVecs>(srow, grow, P, kb, forced_from, sh);
  const int total = got.total;

  // the k-th of them: one wave alone, whose rounds need no barrier
  // (stores at -1 lie outside the buffer and are dropped, which costs less than a branch)
  const __amdgpu_buffer_rsrc_t list = __builtin_amdgcn_make_buffer_rsrc(out, 0, kb * 4, 0x27000);
  auto emit = [&](int, int at, int page) { __builtin_amdgcn_raw_buffer_store_b32(page, list, at * 4, 0, 0); };
  if (wave > 0) return;
  if (total <= 4 * kWave) select_gathered<4>(sh.kept, total, got.T0 - 1u, got.top, kb, emit);
  else if (total <= 8 * kWave) select_gathered<8>(sh.kept, total, got.T0 - 1u, got.top, kb, emit);
  else if (total <= 16 * kWave) select_gathered<16>(sh.kept, total, got.T0 - 1u, got.top, kb, emit);
  else select_gathered<kKept / kWave>(sh.kept, total, got.T0 - 1u, got.top, kb, emit);
}

}  // namespace

hipError_t launch_select_grouped(const CacheView& c, const float* d_scores, const uint32_t* d_group_max, int score_stride,
                                 int top_k, int32_t* d_sel_pages, int32_t* d_sel_count, hipStream_t stream) {
  const int P = c.max_pages_hint;
  if (!select_uses_groups(P, top_k)) return hipErrorInvalidValue;  // the kernels are made for these sizes alone
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
