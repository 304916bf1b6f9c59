// Which dense decodes are cut by the lengths on the device (dense.hip), into how many chunks at most, and how. Whole numbers only (no
// HIP), so that it can be checked without a GPU, and so that the kernel that writes the chunks and the one that merges them, which
// find the cut each for itself, cannot differ. (constexpr functions are compiled for the device, too.)
#pragma once
#include <stdint.h>

#include "split_plan.hpp"

namespace unique {

constexpr int kDenseSlots = 512;    // workgroups that run at the same time: two on each of the 256 compute units
constexpr int kDensePages = 256;    // pages of a chunk from which on twice the workgroups are used
constexpr int64_t kDenseLeastBytes = 96ll << 20;
constexpr int kDenseMaxBatch = 64;  // a lane per sequence

// Chunks of the whole batch, at most as many as the partial results of most_splits hold.
inline int dense_max_chunks(int rows, int max_pages) {
  const int64_t all = (int64_t)rows * most_splits(rows, max_pages).num_splits;
  const int64_t wanted = std::max<int64_t>((int64_t)rows * max_pages / (kDenseSlots * kDensePages), 1) * kDenseSlots;
  return (int)std::min(all, wanted);
}

// Finding the cut costs 0.5 us or more in both kernels, which launches that cannot read 96 MB do not get back (2 sequences of up to 4000
// tokens, 8 KV heads: 12.9 us with most_splits, 14.4 so; 4 of 2048, fp32: 18.9 and 20.5). us of the whole call before / now (bf16,
// 8 KV heads, G = 4, D = 128, pages of 16): 4 sequences of 6K to 30K tokens 66.4 / 43.2; 8 of 2K to 60K, 1012 MB 205 / 163; 16 of 1K
// to 16K 128 / 70; even ones 8 x 16384 86.6 / 86.5, 16 x 30000 312 / 299, 5 x 7000 31.3 / 30.1. More rows than half the slots, and a
// single sequence, have nothing to gain.
inline bool dense_balances(int batch, int kv_heads, int max_pages, int page_bytes) {
  const int64_t rows = (int64_t)batch * kv_heads;
  if (batch < 2 || batch > kDenseMaxBatch || rows > kDenseSlots / 2 || rows * max_pages > INT32_MAX) return false;
  return most_splits((int)rows, max_pages).num_splits > 1 && rows * max_pages * page_bytes >= kDenseLeastBytes;
}

// One wave merges a head's chunks where the slots are four or fewer to a row, on average: every wave finds the cut for itself, which costs more
// than it gains by reading an eighth or so of the rows. kernel us with four / one: 32 x 8 rows of 8 heads, lengths uniform 8.0 / 4.7, 64 x 2 of 8 heads 5.8 / 4.3, 16 x 8
// of 4 heads 4.3 / 4.3 (the call 141.2 / 140.8); 4 x 8 of 8 heads 4.3 / 5.2, 64 x 1 of 8 heads, log-uniform 4.2 / 5.2, 2 x 32 4.3 / 4.6.
constexpr bool dense_merge_alone(int rows) { return rows >= kDenseSlots / 4; }

// Workgroups that share the pages of a batch, `total` of them over all rows: those that run at the same time, or a multiple.
constexpr int dense_slots(int total, int max_chunks) {
  const int rounds = total / (kDenseSlots * kDensePages);
  return std::min((rounds > 1 ? rounds : 1) * kDenseSlots, max_chunks);
}
// Where there is room for a chunk per row beside the slots, rows of less than a quarter of a chunk take only an eighth or two of a slot
// each, as they are soon done: one sequence of 100000 tokens beside 30 of 50, whose 240 rows would leave it half of the slots, 104 / 76
// us. (With all rows of less than a chunk counted by their length 32 sequences of 2118 to 15715 tokens took 228 us instead of 192.)
constexpr bool dense_has_room(int rows, int slots, int max_chunks) { return max_chunks - rows >= slots; }

// The cut: chunks per page as a fraction of 2^32, the same for all rows. It says into how many equal chunks a row is cut.
constexpr uint32_t kDenseMostRate = (1u << 30) - 1;  // a page per wave
constexpr uint32_t dense_eighths(int pages, uint32_t rate) { return (uint32_t)(((uint64_t)((uint32_t)pages * 8u) * rate) >> 32); }
constexpr int dense_row_chunks(int pages, uint32_t rate) { return pages > 0 ? (int)(dense_eighths(pages, rate) / 8u) + 1 : 0; }
constexpr int dense_row_weight(int pages, uint32_t rate, bool room) {  // eighths of a slot
  const uint32_t e = dense_eighths(pages, rate);
  return pages > 0 ? (int)(room && e < 2u ? e + 1u : e / 8u * 8u + 8u) : 0;
}

// The largest rate, within a 64th, at which the rows have no more weight than there are slots; weights(rate): that of all rows. The
// first one is certain to fit, as a row's last chunk is its only one that is not full; no rate above an equal share can. slots > rows.
template <typename Weights>
constexpr uint32_t dense_rate(int total, int rows, int slots, Weights weights) {
  const uint32_t per = 0xffffffffu / (uint32_t)std::max(total, 1);
  uint32_t fits = (uint32_t)std::min<uint64_t>((uint64_t)per * (uint32_t)(slots - rows), kDenseMostRate);
  uint32_t fails = (uint32_t)std::min<uint64_t>(((uint64_t)per + 1) * (uint32_t)slots, 0xffffffffu);
  while (fits < kDenseMostRate && fails - fits > std::max(fits / 64u, 1u)) {
    const uint32_t rate = std::min(fits + (fails - fits) / 2, kDenseMostRate);
    if (weights(rate) <= 8 * slots) fits = rate;
    else fails = rate;
  }
  return fits;
}

// Equally long sequences have as many chunks per row as there is room for, of at least a page per wave.
constexpr int dense_even_chunks(int pages, int rows, int slots) {
  return std::min(slots / rows, (pages + kDecWaves - 1) / kDecWaves);
}

}  // namespace unique
