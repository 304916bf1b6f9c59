// Which selections use the group maxima of the scores, and which decode steps select and attend in one kernel. Host arithmetic on the launch's bounds only (no HIP), so that it can be
// checked without a GPU.
#pragma once
#include <stdint.h>

#include "split_plan.hpp"

namespace unique {

constexpr int kStepMaxPages = 4096;  // pages of a row: 16 scores per thread
constexpr int kStepMaxGroupPages = 32768;  // pages of a row that is selected from by its group maxima: 16 of them per thread
constexpr int kStepMaxTopK = 256;    // list entries that a workgroup keeps in the LDS

constexpr int kStepWholePages = 384;  // pages of a row that are scored in the same kernel, too

constexpr int kGroupsMaxPages = 131072, kGroupsMaxTopK = 1280, kGroupsPagesPerK = 24;  // selections from the group maxima

// Selections of rows whose group maxima the score kernel leaves beside the scores: worth it while the kept groups are a small part of
// the row and fit the workgroup's registers (2048 of them, k and a half and some more). Kernel us of select.hip / select_grouped.hip,
// planted normal scores, 8 rows: 4097 pages, k 64 7.8 / 5.9; 8192, 64 8.6 / 5.4; 12000, 500 11.9 / 9.0; 16384, 64 9.7 / 6.8; 32768, 64
// 13.9 / 7.6; 62501, 1024 29.6 / 14.1; 64 rows: 8192, 256 8.9 / 7.3; 128 rows: 16384, 680 13.5 / 11.0; 16 rows: 125001, 1024 45.2 /
// 19.3. Not worth it: 4097, 340 7.6 / 7.7; 16384, 1024 (128 rows) 14.0 / 16.4. The maxima cost the score kernel 0.3 us (1 us of 90 at
// 16 x 16384 pages).
// Scores that rise by two standard deviations along the row need a tighter bound and take longer, not longer than there but where k
// is near its limit: 4097, 64 7.8 / 7.4; 8192, 256 8.4 / 9.3; 12000, 500 11.4 / 11.9; 16384, 680 12.8 / 14.4; 62501, 1024 28.7 /
// 17.0. Scores of five values: 8192, 256 19.4 / 8.0; 62501, 1024 40.8 / 17.7; 125001, 1024 431 / 26.5.
inline bool select_uses_groups(int max_pages, int top_k) {
  return max_pages > kStepMaxPages && max_pages <= kGroupsMaxPages && top_k <= std::min(max_pages / kGroupsPagesPerK, kGroupsMaxTopK);
}

// Saved are a launch and the round trips of writing and reading the list, paid is a selection by four waves in every
// workgroup of a cut row. us of a whole step in separate kernels / so (bf16, 8 KV heads, G = 4, D = 128, pages of 16, fp32 means):
//   1 x 2048 pages, k = 128 22.2 / 19.7; 1 x 4096, 64 22.7 / 19.7; 8 x 1000, 64 25.3 / 22.3; 40 x 64, 8 20.6 / 18.6;
//   80 x 1000, 64 124.7 / 121.1 (uncut rows)
// From some k on too many keys are gathered: 1 x 2048, 512 25.5 / 28.6; 1 x 1000, 300 23.1 / 24.2 (a bound on the k-th key needs
// more than k groups of four pages; up to 512 pages it does not matter: 8 x 250, 200 34.0 / 32.4).
// Workgroups that wait for a free unit select when the others already stream: 24 x 1000 pages cut in 5, 960 workgroups, 48.6 /
// 47.2. The longer the rows, the fewer workgroups they are cut into: 1024 up to 2048 pages, 512 at 4096, in between as many as read that many scores;
// but always 768 where three_fit, k = 128 in separate kernels / so: 20 x 4096 (640 workgroups) bf16 means 75.0 / 72.7, fp32 means 101.1 / 98.9, 17 x 4096, k = 64
// (544) 53.6 / 49.1, 31 x 4096, 64 121.5 / 115.3, 30 x 3000 (720) 90.4 / 86.6, 28 x 4064 (672) of D = 64 60.9 / 59.1, G = 8 102.5 / 97.9, pages of 32 96.4 / 89.3, of an fp32 cache, pages of 8
// 132.8 / 131.6, lengths from a 20th of the longest 71.4 / 67.9. bf16 caches of 128 channels in pages of 8 have room for two: 20 x 4095, k = 256 104.6 /
// 107.2, G = 8 81.2 / 83.6 (k = 128 gains at every length, 20 x 2100 50.8 / 49.9, 20 x 4000 62.6 / 62.0; k = 256 at none, 20 x 2600 65.9 / 66.8). Rows selected from their group maxima stay at 512: 17 x 5000 101.9 / 103.9, 22 x 6000 108.8 / 109.0.
// Longer rows, from their group maxima, in kernels of their own (select_grouped.hip) / so: 1 x 4200, 64 24.8 / 22.1; 1 x 8192, 256 29.0 /
// 27.8; 16 x 8192, 256 143.8 / 141.8; 1 x 32768, 128 41.7 / 40.0; 4 x 16384, 64 62.9 / 60.7. Scores that rise by two standard deviations
// along the row, with a selection that reads every score / so: 1 x 8192, 256 27.7 / 28.3; 16 x 8192, 256 141.4 / 142.6; 1 x 4200, 64
// 22.2 / 22.0; 4 x 16384, 64 63.0 / 60.4; 1 x 32768, 256 47.9 / 43.9.
inline bool step_fuses(int rows, int max_pages, int top_k, const SplitPlan& plan, bool three_fit = false) {
  if (max_pages > kStepMaxGroupPages || top_k > kStepMaxTopK || (max_pages > 512 && 4 * top_k > max_pages)) return false;
  if (max_pages > kStepMaxPages) return select_uses_groups(max_pages, top_k) && (plan.num_splits == 1 || (int64_t)rows * plan.num_splits <= 512);
  const int most = std::max(1024 * 2048 / std::max(max_pages, 2048), three_fit ? 768 : 0);
  return plan.num_splits == 1 || (int64_t)rows * plan.num_splits <= most;
}

// Kernels that select and attend whose registers are held down to what leaves a unit room for three workgroups (step.hip): bf16 caches of 128
// channels take just more than a third of them when left alone. 24 x 1000 pages, k = 64, 960 workgroups, 34.9 us, so 32.6, 100 x 1000, 32
// 81.8 / 80.3, launches that fit either way the same. Pages of 8 tokens would need scratch memory for it.
constexpr bool step_held(bool bf16, int head_dim, int page_size) { return bf16 && head_dim == 128 && page_size >= 16; }
// Whether cut rows may have as many workgroups as three to a unit are: the held kernels have room for them, and so have the others but bf16
// caches of 128 channels in pages of 8, and eight heads of an fp32 cache of 128 channels, which gain all the same, as their attention is bound by
// arithmetic. us in separate kernels / so, fp32, G = 8, k = 128: 20 x 4000 pages of 8 89.5 / 87.6, of 16 124.0 / 122.9, of 32 189.5 / 189.0; of 16 17 x 4096,
// 64 85.1 / 83.4, 31 x 4096, 64 125.2 / 122.8, 31 x 2732 150.8 / 152.0; of 32 24 x 3000, 64 140.3 / 137.8, 20 x 2200, 256 307.9 / 307.8.
constexpr bool step_three_fit(bool bf16, int head_dim, int page_size) { return !bf16 || head_dim != 128 || step_held(bf16, head_dim, page_size); }

// LDS that a launch of the held kernels adds to their own, so that only two of its workgroups find a place on a unit. Where rows are not cut and their
// lists are long, three to a unit take a third longer each, and of rows of unlike lengths the long ones end on few units; two leave more rows
// to the units that are done. By the bytes of K and V of a list, us with three / two (pages of 16, lengths log-uniform from a 20th, or one long and the
// others a quarter or a tenth): 128 KB 180 x 300 pages 49.7 / 53.2, 256 KB 100 x 1000 58.6 / 60.0, 384 KB 110 x 171 59.1 / 60.3, G = 8 120 x 300 50.8 /
// 52.5; 512 KB 80 x 300 66.1 / 62.7, G = 8 75 x 300 49.7 / 43.5, but G = 1 70 x 500 65.8 / 70.8; 768 KB 90 x 300 53.1 / 46.7; 1 MB G = 2 132 x 700 181 /
// 169; 2 MB G = 1 83 x 500 148 / 121; 4 MB G = 2 70 x 300 393 / 354. Even batches are the same from 512 KB on (75 x 300 129.6 / 128.9).
constexpr int64_t kStepLongList = 512 << 10;
constexpr int step_extra_lds(bool held, int num_splits, int64_t list_bytes, int own_bytes) {
  constexpr int kTwoFit = 56 << 10;  // more than a third of a unit's LDS
  return held && num_splits == 1 && list_bytes >= kStepLongList ? std::max(kTwoFit - own_bytes, 0) : 0;
}

// Steps whose rows are so short that every workgroup of a row's chunks scores the row for itself: one launch, at most with a merge
// behind it. us of a whole step, three or four kernels / two or three / so (bf16, 8 KV heads, G = 4, D = 128, pages of 16, fp32 means):
//   1 x 64 pages, k = 8 15.5 / 13.9 / 10.8; 1 x 128, 64 18.3 / - / 13.5; 16 x 128, 16 17.9 / 16.4 / 13.3; 80 x 64, 8 26.2 / 25.0 / 24.3;
//   1 x 250, 200 19.9 / 19.5 / 17.3; the toy model (2 heads, fp32, D = 64, 128 pages, k = 16) 14.9 / 13.5 / 11.4
// Reading a row's means takes one compute unit longer than a launch costs from 128 KB on: 16 x 270 pages 18.4 / 15.8, but 4 x 320,
// k = 64 18.7 / 20.5 and 4 x 512, 64 19.1 / 23.2; rows of 256 bytes: 2 x 400, 16 heads, G = 8 21.8 / 20.4, 6 x 500, G = 1 21.6 / 20.0,
// 10 x 500, G = 8 21.0 / 22.2. Cut rows of more workgroups than run at the same time score their rows once more in a second round: 24 x
// 250, 64 (576 workgroups) three kernels 36.5, so 42.0; 17 x 250, 48 28.9 / 33.9; 20 x 120, 64 31.1 / 32.1; 28 x 250, 64 41.7 / 41.5.
inline bool step_is_whole(int rows, int max_pages, int mean_bytes, bool streams, const SplitPlan& plan) {
  if (plan.num_splits > 1 && (int64_t)rows * plan.num_splits > 512) return false;
  return max_pages <= (mean_bytes > 256 ? 256 : kStepWholePages) && !streams;
}

}  // namespace unique
