// C interface of the launch rules for the CPU tests.
#include <cmath>
#include <cstdlib>

#include "../../paper_2605_27740_amd/csrc/dense_plan.hpp"
#include "../../paper_2605_27740_amd/csrc/score_tile.hpp"
#include "../../paper_2605_27740_amd/csrc/split_plan.hpp"
#include "../../paper_2605_27740_amd/csrc/stats_bulk.hpp"
#include "../../paper_2605_27740_amd/csrc/step_rule.hpp"

extern "C" void most(int rows, int len, int* out) {
  const unique::SplitPlan p = unique::most_splits(rows, len);
  out[0] = p.pages_per_split; out[1] = p.num_splits; out[2] = p.rotate;
}
extern "C" void plan(int batch, int kv_heads, int len, int max_pages, int page_bytes, int slow, int* out) {
  const unique::SplitPlan p = unique::plan_splits(batch, kv_heads, len, max_pages, page_bytes, slow != 0);
  out[0] = p.pages_per_split; out[1] = p.num_splits; out[2] = p.rotate;
}
extern "C" int tile(int batch, int kv_heads, int head_dim, int max_pages, int min_pages, int max_tile) {
  return unique::score_tile(batch, kv_heads, head_dim, max_pages, min_pages, max_tile);
}
extern "C" int even_tile(int tile, int batch, int max_pages, int min_pages, int mean_bytes, int max_tile) {
  return unique::score_even_tile(tile, batch, max_pages, min_pages, mean_bytes, max_tile);
}
extern "C" int last_page_rule(int cut, int workgroups, int last_pages, int mb, int group, int fitted) {
  return unique::score_last_page_rule(cut != 0, workgroups, last_pages, (int64_t)mb << 20, group, fitted != 0);
}
extern "C" void score_grid(int cut, int tiles, int batch, int kv_heads, long long bytes, int group, int fitted, int* out) {
  const unique::ScoreGrid g = unique::score_grid(cut != 0, tiles, batch, kv_heads, true, bytes, group, fitted != 0);
  out[0] = g.x, out[1] = g.y, out[2] = g.refresh & ((1 << unique::kLastPageBits) - 1), out[3] = g.refresh >> unique::kLastPageBits;
}
extern "C" int tile_stride(int tile) { return unique::score_tile_stride(tile); }
extern "C" int bulk(long long record_bytes, int head_dim, int page_size, int key_bytes, int bf16_means) {
  return unique::stats_bulk(record_bytes, head_dim, page_size, key_bytes, bf16_means != 0);
}
extern "C" int fuses(int batch, int kv_heads, int max_pages, int top_k, int page_bytes) {
  return unique::step_fuses(batch * kv_heads, max_pages, top_k,
                            unique::plan_splits(batch, kv_heads, top_k, max_pages, page_bytes, false));
}
extern "C" int fuses_of(int batch, int kv_heads, int max_pages, int top_k, int page_size, int head_dim, int bf16) {
  return unique::step_fuses(batch * kv_heads, max_pages, top_k,
                            unique::plan_splits(batch, kv_heads, top_k, max_pages, page_size * head_dim * (bf16 ? 4 : 8), false),
                            unique::step_three_fit(bf16 != 0, head_dim, page_size));
}
extern "C" int extra_lds(int bf16, int head_dim, int page_size, int num_splits, long long list_bytes, int own_bytes) {
  return unique::step_extra_lds(unique::step_held(bf16 != 0, head_dim, page_size), num_splits, list_bytes, own_bytes);
}
extern "C" int whole(int batch, int kv_heads, int max_pages, int top_k, int page_bytes, int mean_bytes, int streams) {
  return unique::step_is_whole(batch * kv_heads, max_pages, mean_bytes, streams != 0,
                               unique::plan_splits(batch, kv_heads, top_k, max_pages, page_bytes, false));
}
extern "C" int uses_groups(int max_pages, int top_k) { return unique::select_uses_groups(max_pages, top_k); }
extern "C" int dense_chunks(int rows, int max_pages) { return unique::dense_max_chunks(rows, max_pages); }
extern "C" int dense_balances(int batch, int kv_heads, int max_pages, int page_bytes) {
  return unique::dense_balances(batch, kv_heads, max_pages, page_bytes);
}
extern "C" int lds(int scores, int elem_bytes, int head_dim, int group, int workgroups) {
  return unique::score_lds(scores, elem_bytes, head_dim, group, workgroups);
}
// The cut of a dense batch as dense.hip finds it: chunks per row of every sequence; returns the workgroups that look for a chunk.
extern "C" int dense_cut(const int* pages, int batch, int kv_heads, int max_pages, int* chunks) {
  const int rows = batch * kv_heads, max_chunks = unique::dense_max_chunks(rows, max_pages);
  int total = 0;
  bool even = true;
  for (int b = 0; b < batch; ++b) {
    total += pages[b] * kv_heads;
    even = even && pages[b] == pages[0];
  }
  const int slots = unique::dense_slots(total, max_chunks);
  const bool room = unique::dense_has_room(rows, slots, max_chunks);
  const uint32_t rate = unique::dense_rate(total, rows, slots, [&](uint32_t r) {
    int weight = 0;
    for (int b = 0; b < batch; ++b) weight += unique::dense_row_weight(pages[b], r, room);
    return weight * kv_heads;
  });
  for (int b = 0; b < batch; ++b)
    chunks[b] = even ? unique::dense_even_chunks(pages[b], rows, slots) : unique::dense_row_chunks(pages[b], rate);
  return room ? slots + rows : slots;
}
extern "C" int score_cuts(int batch, int max_pages, int min_pages, int mean_bytes, long long rec_bytes) {
  return unique::score_cuts(batch, max_pages, min_pages, mean_bytes, rec_bytes);
}
extern "C" int held_lds(int elem_bytes, int head_dim, int group) { return unique::score_held_lds(elem_bytes, head_dim, group); }
extern "C" int dense_merge_alone(int rows) { return unique::dense_merge_alone(rows); }
extern "C" int score_cut_reserve(int batch, int kv_heads, long long bytes, int group, int head_dim, int bf16_means) {
  return unique::score_cut_reserve(true, batch, kv_heads, bytes, group, unique::score_cut_two_fit(group, head_dim, bf16_means != 0));
}
extern "C" int score_cut_three_fit(int group, int head_dim, int bf16_means, int elem_bytes, int batch) {
  return unique::score_cut_three_fit(group, head_dim, bf16_means != 0, elem_bytes, batch);
}
extern "C" int score_cut_grid(int batch, int max_pages, int most_pages, int three_fit, int reserve) {
  return unique::score_cut_grid(batch, max_pages, most_pages, three_fit != 0, reserve);
}
// The cut of a batch's scores as score.hip finds it: chunks of every sequence and the units of each of them; returns the pages of a chunk at
// most. The reciprocals are `ulps` units in the last place off.
extern "C" int score_cut(const int* pages, int batch, int most_pages, int three_fit, int reserve, int ulps, int* chunks, int* sizes) {
  const int most = most_pages / unique::kCutUnit;
  auto units = [&](int b) { return (pages[b] + unique::kCutUnit - 1) / unique::kCutUnit; };
  auto reciprocal = [&](int n) {
    float r = 1.f / (float)n;
    for (int i = 0; i < std::abs(ulps); ++i) r = std::nextafter(r, ulps < 0 ? 0.f : 2.f);
    return r;
  };
  int all = 0;
  for (int b = 0; b < batch; ++b) all += units(b);
  const int slots = unique::score_cut_slots(all, batch, most, three_fit != 0, reserve);
  int chunk = 0;
  for (int waste : {batch / 2, batch}) {
    chunk = unique::score_cut_chunk(all, slots, waste, most);
    int sum = 0;
    for (int b = 0; b < batch; ++b) sum += chunks[b] = unique::score_cut_chunks(units(b), chunk, reciprocal(chunk));
    if (sum <= slots) break;
  }
  for (int b = 0; b < batch; ++b) sizes[b] = chunks[b] > 0 ? unique::score_cut_chunks(units(b), chunks[b], reciprocal(chunks[b])) : 0;
  return chunk * unique::kCutUnit;
}
