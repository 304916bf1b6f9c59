// How the page lists of a decode launch are cut into chunks, one workgroup each. Host arithmetic on the launch's bounds
// only (no HIP), so that it can be checked without a GPU.
#pragma once
#include <stdint.h>

#include <algorithm>

namespace unique {

constexpr int kDecWaves = 4;  // waves of a decode workgroup

struct SplitPlan {
  int32_t pages_per_split;  // list entries handled by one workgroup
  int32_t num_splits;       // grid extent along the split axis (upper bound for every row)
  int32_t rotate;           // 0: grid (split, head, sequence). Else a power of two <= batch: grid (head, sequence, split)
};

// Partial results are sized for this many chunks per row, the most that any launch below cuts a list into.
inline SplitPlan most_splits(int rows, int max_list_len) {
  constexpr int64_t kGroups = 512, kMaxPages = 256;
  rows = std::max(rows, 1);
  const int64_t len = std::max(max_list_len, 1);
  const int64_t wanted = rows >= 256 ? 1 : (kGroups + rows - 1) / rows;
  int64_t pps = std::max<int64_t>((len + wanted - 1) / wanted, kDecWaves);  // at least one page per wave
  // long lists are cut into many equal chunks so that ragged batches balance across the CUs
  pps = (std::min(pps, kMaxPages) + kDecWaves - 1) / kDecWaves * kDecWaves;
  return SplitPlan{(int32_t)pps, (int32_t)((len + pps - 1) / pps), 0};
}

// Lists of a selection or of a caller, of which only an upper bound on the length is known here. us of the partial and merge
// kernels on data that is not in the caches, G = 4, pages of 8 KB.
// Most rows are as long as max_list_len says, and a cut that gives the compute units equal shares is then best: what the
// busiest of the 256 units has to read bounds the launch, ceil(workgroups / 256) chunks; below 1.2 times the average share
// the memory bounds it, below 64 KB latency, and the merge launch that every cut row needs costs as much as 160 KB.
// Candidates are an uncut row, the largest numbers of chunks that fill one to four workgroups per unit, and the cut of
// most_splits, which only a clear gain gives up for more than one workgroup per unit:
//   96 rows x 200 pages: 5 chunks 32.4 (6, most_splits: 38); 16 x 1024: 16 chunks 29.2 (32: 31)
//   160 x 32: uncut 12.0 (4 chunks 17.4); 16 x 16: uncut 6.3 (4 chunks 8.0)
// But rows may be shorter, and a long row among short ones takes as long as its longest chunk, which a unit reads at 35 KB
// per us. A chunk may therefore be 256 KB longer than that of most_splits, no more (one list of eight full, the others a
// sixteenth of it; all equal shares / this rule): 192 x 150 pages 37.0 / 20.7, 128 x 256 35.7 / 25.8, 256 x 1024 232 / 83.
// With that bound no mixture of lengths measured slower than most_splits but one: 16 rows of 50 to 60 entries in lists of
// 600, 14.5 against 13.6. It costs full lists that would be better uncut: 192 x 150 pages 52.4 instead of 47.6.
// slow_arithmetic (8 query heads on the vector units, fp32 caches): a workgroup alone on its unit takes 1.2 us for a page per
// wave, so a row goes uncut only 64 KB beyond the cut of most_splits. 8 rows x 16 pages of 8 KB: uncut 11.3, 4 chunks 9.5.
// Where all entries that can be pages fit one chunk of most_splits, cutting the rest off gains nothing.
// Lists longer than the sequences have pages and cut lists of 256 rows or more always have empty chunks, and these come last
// (SplitPlan::rotate): as the fastest grid index they are a regular subset of the workgroups, which leaves whole XCDs and
// compute units without work. 32 rows x 125 of 1024 pages: 35.1 split first, 21.7 split last; 64 x 256 of 1024: 65.2 and
// 38.8; 256 rows of 100 to 2000 entries in lists of 8192: 1590 and 296.
inline SplitPlan plan_splits(int batch, int kv_heads, int max_list_len, int max_pages, int page_bytes,
                             bool slow_arithmetic) {
  constexpr int64_t kCUs = 256, kMergeBytes = 160 << 10, kLeastBytes = 64 << 10, kMoreBytes = 256 << 10, kMaxGridZ = 65535;
  const int rows = std::max(batch * kv_heads, 1);
  const SplitPlan most = most_splits(rows, max_list_len);
  const int64_t len = std::max(max_list_len, 1), filled = std::min<int64_t>(len, max_pages);
  const int64_t longest = most.pages_per_split + kMoreBytes / page_bytes;
  const int64_t longest_uncut = most.pages_per_split + (slow_arithmetic ? kMoreBytes / 4 : kMoreBytes) / page_bytes;
  auto cost_of = [&](int64_t pps) {
    const int64_t share = (rows * ((filled + pps - 1) / pps) + kCUs - 1) / kCUs * std::min(pps, filled) * page_bytes;
    return std::max({share, rows * filled * page_bytes / kCUs * 6 / 5, kLeastBytes}) + (pps < len ? kMergeBytes : 0);
  };
  const int64_t most_cost = cost_of(most.pages_per_split);
  SplitPlan best = most;
  int64_t best_cost = most_cost;
  for (int w = 0; w <= 4; ++w) {
    const int64_t s = w == 0 ? 1 : std::min<int64_t>(kCUs * w / rows, most.num_splits);
    if (s < 1) continue;
    const int64_t pps = ((len + s - 1) / s + kDecWaves - 1) / kDecWaves * kDecWaves;
    const int64_t n = (len + pps - 1) / pps, cost = cost_of(pps);
    const bool fits = n == 1 && filled <= most.pages_per_split && len <= 4 * most.pages_per_split;
    if ((pps > (n == 1 ? longest_uncut : longest) && !fits) || n > most.num_splits || (w > 1 && cost * 10 > most_cost * 9)) continue;
    if (cost < best_cost || (w <= 1 && best_cost == most_cost && cost == most_cost)) {
      best = SplitPlan{(int32_t)pps, (int32_t)n, 0};
      best_cost = cost;
    }
  }
  if (best.num_splits > 1 && best.num_splits <= kMaxGridZ && (len > max_pages || rows >= kCUs))
    for (best.rotate = 1; best.rotate <= batch / 2;) best.rotate *= 2;
  return best;
}

}  // namespace unique
