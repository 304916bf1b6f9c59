// Internal launch interface between the C ABI (api.hip) and the kernel translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "split_plan.hpp"

namespace unique {

// Device pointers and dimensions of the paged cache, passed by value to every kernel. Aligned so that the arguments behind it
// start on a 16-byte boundary and are fetched whole (the merge kernel of one 32K sequence takes 4.34 us 8 bytes further on, 4.12 so).
struct alignas(16) CacheView {
  const void* k_cache;        // [num_phys][Hkv][S][D]
  const void* v_cache;
  void* page_stats;           // [num_phys] records: Hkv*D means (fp32 or bf16), Hkv fp32 stds, pad to kStdBlockBytes
  const int32_t* page_table;  // [B][max_pages]
  const int32_t* seq_lens;    // [B]
  int32_t H, Hkv, D, S, B, max_pages;
  int64_t num_phys;
  int32_t dtype;              // 0 fp32, 1 bf16
  int32_t max_pages_hint;     // host bound on pages of any sequence (<= max_pages)
  int32_t min_pages_hint;     // host lower bound on full pages of every sequence (0: unknown); sizes tiles only
  int32_t stats_bf16;         // 1: means stored as bf16, 0: fp32
  int64_t rec_bytes;          // bytes per page record of page_stats
  int64_t kv_page_stride;     // elements between consecutive physical pages of k_cache (and of v_cache)
  int64_t kv_head_stride;     // elements between consecutive KV heads inside a page
  int32_t force_recent;       // the last this-many logical pages of a sequence are always selected (0: none)
};

// Launches that stream more than this many bytes bypass cache allocation (the Infinity Cache holds 256 MB).
constexpr int64_t kStreamNtBytes = 96ll << 20;

constexpr int kStdBlockBytes = 128;     // bytes reserved after the means of a page record (fp32 stds + pad)
constexpr int kScoreStrideAlign = 64;  // score rows in the workspace are padded to this many floats
constexpr int kGroupPages = 8;         // consecutive pages that share an entry of the group maxima

bool stats_supported(int dtype, int D, int S);
bool score_supported(int dtype, int D, int G, int Hkv);
bool decode_supported(int dtype, int D, int S, int G);

hipError_t launch_stats(const CacheView& c, const int32_t* d_tok_begin, const int32_t* d_tok_end,
                        int max_pages_touched, hipStream_t stream);

// refresh_tail: the statistics of the last page of every sequence are recomputed from the keys (the same arithmetic as launch_stats) and
// stored before that page is scored; d_scores_out is null then. d_group_max may then not count a last page that is scored apart from its group: whoever reads the
// maxima takes that page's score itself.
// d_group_max: [rows][score_stride / kGroupPages], the largest key (score_key) of every group of pages; null: not wanted.
hipError_t launch_score(const CacheView& c, const void* d_q, float lambda, float* d_scores, int score_stride,
                        float* d_scores_out, uint32_t* d_group_max, bool refresh_tail, hipStream_t stream);

// d_group_max: of the same scores, where select_uses_groups (step_rule.hpp) wants them, or null
hipError_t launch_select(const CacheView& c, const float* d_scores, const uint32_t* d_group_max, int score_stride, int top_k,
                         int32_t* d_sel_pages, int32_t* d_sel_count, hipStream_t stream);

// The selection for rows whose group maxima are known, which reads only the groups that can hold a selected page
// (select_uses_groups in step_rule.hpp says for which launches).
hipError_t launch_select_grouped(const CacheView& c, const float* d_scores, const uint32_t* d_group_max, int score_stride,
                                 int top_k, int32_t* d_sel_pages, int32_t* d_sel_count, hipStream_t stream);

// d_sel_pages == nullptr: attend every page of each sequence (dense).
hipError_t launch_decode(const CacheView& c, const void* d_q, const int32_t* d_sel_pages,
                         const int32_t* d_sel_count, int sel_stride, int max_list_len, float sm_scale,
                         void* d_out, float* d_lse_out, float* d_partials, hipStream_t stream);

// Attention over the page lists of a selection and the merge of its chunks: what launch_decode does for the list d_sel_pages
// of stride top_k, as the plan, the arguments and the parts that launch_select_decode shares with it.
struct StepArgs {
  const void* q;
  const float* scores;   // [rows][score_stride]; null: the kernel scores the pages, too (step_is_whole)
  const uint32_t* group_max;  // of those scores, for rows of more than kStepMaxPages pages
  int score_stride, top_k;
  float lambda;          // of those scores
  int refresh_tail;
  int32_t* sel_pages;
  int32_t* sel_count;
  float sm_scale;
  void* out;
  float* lse_out;
  float* partials;       // must not overlap the scores
};
SplitPlan selection_plan(const CacheView& c, int top_k);
size_t plan_partial_floats(const CacheView& c, const SplitPlan& plan);
bool decode_streams(const CacheView& c, int max_list_len);  // K and V are read with non-temporal loads
float decode_scale_log2(const CacheView& c, float sm_scale);
hipError_t launch_merge(const CacheView& c, const int32_t* d_sel_count, int sel_stride, const SplitPlan& plan, float* d_partials,
                        void* d_out, float* d_lse_out, hipStream_t stream);

// Selection and attention in one kernel (step_rule.hpp says for which steps); a cut row needs launch_merge behind it.
template <typename T, int D, int S>
hipError_t launch_select_decode(const CacheView& c, const StepArgs& a, hipStream_t stream);
#define UNIQUE_DECLARE(T, D, S) template <> hipError_t launch_select_decode<T, D, S>(const CacheView&, const StepArgs&, hipStream_t);
#define UNIQUE_DECLARE_PAGES(T, D) UNIQUE_DECLARE(T, D, 8) UNIQUE_DECLARE(T, D, 16) UNIQUE_DECLARE(T, D, 32)
UNIQUE_DECLARE_PAGES(float, 64) UNIQUE_DECLARE_PAGES(float, 128) UNIQUE_DECLARE_PAGES(uint16_t, 64) UNIQUE_DECLARE_PAGES(uint16_t, 128)
#undef UNIQUE_DECLARE_PAGES
#undef UNIQUE_DECLARE

// Attention over every page, cut by the lengths on the device (dense_plan.hpp says for which launches).
template <typename T, int D>
hipError_t launch_dense(const CacheView& c, const void* d_q, float sm_scale, void* d_out, float* d_lse_out, float* d_partials,
                        hipStream_t stream);
template <> hipError_t launch_dense<float, 64>(const CacheView& c, const void* d_q, float sm_scale, void* d_out, float* d_lse_out,
                                         float* d_partials, hipStream_t stream);
template <> hipError_t launch_dense<float, 128>(const CacheView& c, const void* d_q, float sm_scale, void* d_out, float* d_lse_out,
                                         float* d_partials, hipStream_t stream);
template <> hipError_t launch_dense<uint16_t, 64>(const CacheView& c, const void* d_q, float sm_scale, void* d_out, float* d_lse_out,
                                         float* d_partials, hipStream_t stream);
template <> hipError_t launch_dense<uint16_t, 128>(const CacheView& c, const void* d_q, float sm_scale, void* d_out, float* d_lse_out,
                                         float* d_partials, hipStream_t stream);

// floats of split-K partial storage needed for a list of at most max_list_len pages per row
size_t decode_partial_floats(const CacheView& c, int max_list_len);

}  // namespace unique
