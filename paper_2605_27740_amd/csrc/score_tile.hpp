// Pages per workgroup of the page-score kernel, and workgroups per compute unit. Host arithmetic on the launch's bounds only (no HIP), so that it can be
// checked without a GPU.
#pragma once
#include <stdint.h>

#include <algorithm>

namespace unique {

// Small tiles balance ragged batches and small launches over the 256 CUs; larger ones save prologues (fewer, longer
// streams). From 32 pages on a tile is doubled while the batch is KNOWN to supply enough FULL tiles of the larger size
// (min_pages: a lower bound on the pages of every sequence), or the launch has workgroups to spare whatever the lengths are.
// Enough is two per compute unit. kernel us with tiles of 32 / 64 / 128 / 256 pages, 8 heads, G = 4, not in the caches:
//   4 x 4096 pages, D = 128, bf16 means 10.0 / 11.5 / 17.1 / 28.6; 4 x 8192 18.1 / 16.0 / 18.1 / 28.6; fp32 means 24.4 / 24.5 /
//   24.0 / 33.4; 8 x 8192, D = 64, bf16 means 18.0 / 17.0 / 18.2 / 26.6; 30 x 3000, fp32 means 63.5 / 63.7 / 62.9 / 70.2
// One per unit is enough where the smaller tiles need a second round (D = 128: three workgroups fit a unit, D = 64: five to
// seven), and for up to 128 pages of a single head, of which a wave takes 8 at a time:
//   1 x 50000, D = 128, bf16 means 22.2 / 23.4 / 23.1 / 21.9 (26.1 with two records in flight); 3 x 9000 17.7 / 15.1 / 20.0;
//   4 x 4096 pages of one head, G = 8, fp32 means 7.7 / 6.0 / 6.7 / 8.6
// max_tile: what a wave can hold the page ids of.
inline int score_tile(int batch, int kv_heads, int head_dim, int max_pages, int min_pages, int max_tile) {
  constexpr int kMinTile = 8, kNumCUs = 256, kOneRound = 3 * kNumCUs;
  constexpr int kFatGrid = 4096;  // workgroups above which a launch can afford the next larger tile
  auto tiles = [&](int tile) { return (int64_t)batch * (((int64_t)max_pages + tile - 1) / tile); };
  int tile = 32;
  while (2 * tile <= max_tile) {
    const bool one = (head_dim == 128 && tiles(tile) > kOneRound) || (kv_heads == 1 && tile <= 64);
    if ((int64_t)batch * (min_pages / (2 * tile)) < (one ? kNumCUs : 2 * kNumCUs) && tiles(2 * tile) < kFatGrid) break;
    tile *= 2;
  }
  // a launch too small to give every CU a workgroup is all latency: shorter tiles spread it over more CUs
  // (one sequence of 32K tokens: 10.7 us with 32-page tiles, 8.7 us with 8-page tiles)
  while (tile > kMinTile && tiles(tile) < kNumCUs) tile /= 2;
  return tile;
}

// Bytes of LDS with which a launch of so many workgroups of the page-score kernel gives each: `scores` of them are used, the rest
// keeps the number of workgroups on a compute unit down where the registers would allow one more. The units are dealt the
// workgroups of a launch in turn for as long as all fit, and with sequences whose lengths are regular the full tiles then meet on a
// few of them, while a launch that has to wait for slots fills those that empty tiles have left. us with one workgroup more / so, 8
// heads, G = 4, D = 128, bf16, fp32 means, the other sequences a quarter as long as the first: 16 x 8192 pages 49.1 / 40.7, 16 x 4096
// 27.3 / 22.6, 4 x 32768 55.9 / 48.1; bf16 means, 16 x 8192 28.4 / 22.9; fp32 queries, G = 1, D = 64, 16 x 4096 of 16 heads 27.0 /
// 24.2. Lengths drawn at random from a wide range 17.0 / 14.8 (8 x 166 to 4096), from a narrow one 13.0 / 15.0 (8 x 645 to 4096). A launch
// that does not fit either way is better with more: 8 x 646 to 16384 30.8 / 31.7, 32 x 71 to 2048 21.3 / 21.9. Even batches are
// the same, and so are the shapes that are not named, whose registers allow no more.
inline int score_lds(int scores, int elem_bytes, int head_dim, int group, int64_t workgroups) {
  constexpr int kLds = 160 << 10, kNumCUs = 256;
  int most = 0;  // workgroups per unit; 0: what the registers allow
  if (elem_bytes == 2 && head_dim == 128 && group == 4) most = 3;
  if (elem_bytes == 4 && head_dim == 64 && group <= 2) most = group == 1 ? 7 : 6;
  // Smaller launches fit either way. (Slightly larger ones still fit, as empty tiles leave early: 12 x 196 to 3125 pages, 1176
  // workgroups, 16.8 / 14.9.)
  if (most == 0 || workgroups <= most * kNumCUs || workgroups > (most + 1) * kNumCUs * 5 / 4) return scores;
  return std::max(scores, kLds / (most + 1) + 1024);
}

}  // namespace unique
