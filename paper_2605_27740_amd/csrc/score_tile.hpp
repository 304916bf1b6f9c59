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

// The tile of a batch that is known to be even, or nearly, and has no more workgroups than run at the same time: not a power of two but
// a multiple of 8 pages with which the workgroups are just below a multiple of the units, as the unit with the most pages bounds the
// launch. What a unit needs in flight is one workgroup of rows of 512 bytes, two of 256, three of 128 (tile of score_tile for 6 x 2500 pages
// of 16 heads, D = 64, fp32: 32 pages, 474 workgroups, 14.0 us; 64, 240, 16.7). kernel us with that tile / so (8 heads, D = 128, G = 4, fp32
// means unless it says otherwise): 1 x 9000 pages 11.1 / 9.4, 1 x 20000 19.4 / 17.9, 5 x 2000 11.6 / 10.2, 60 x 300 18.6 / 16.8, 12 x 3125 30.3 /
// 27.1 (G = 8 34.0 / 28.3), 10 x 8192 58.1 / 55.4, 80 x 1000 57.7 / 54.4; bf16 means 1 x 33000 17.9 / 16.2, 100 x 500 21.6 / 20.9, D = 64 24 x 1700
// 11.7 / 11.3; one head, G = 8 4 x 5000 6.2 / 5.7. 50 x 1282 52.9 / 44.4; G = 8 33 x 2132 64.7 / 50.1.
// Where the busiest unit gains less than a twentieth the tile stays.
inline int score_even_tile(int tile, int batch, int max_pages, int min_pages, int mean_bytes, int max_tile) {
  constexpr int kNumCUs = 256, kUnit = 8;
  if (min_pages < max_pages - max_pages / 8) return tile;
  auto busiest = [&](int t) { return ((int64_t)batch * ((max_pages + t - 1) / t) + kNumCUs - 1) / kNumCUs * t; };
  int best = tile;
  // (three where registers leave room for two: 150 x 30, G = 8 8.6 / 10.2)
  for (int per_unit = mean_bytes >= 512 ? 1 : (mean_bytes >= 256 ? 2 : 3); per_unit <= (mean_bytes >= 256 ? 2 : 3); ++per_unit) {
    const int tiles = kNumCUs * per_unit / batch;  // of a sequence
    if (tiles < 1) continue;
    const int64_t t = ((max_pages + tiles - 1) / tiles + kUnit - 1) / kUnit * kUnit;
    if (t <= max_tile && busiest((int)t) * 20 < busiest(best) * 19) best = (int)t;
  }
  return best;
}
// Scores between two heads of a tile in the LDS.
constexpr int score_tile_stride(int tile) {
  int stride = 8;
  while (stride < tile) stride *= 2;
  return stride;
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

// bf16 caches of 64 channels leave room for one workgroup more than this, which costs batches with empty tiles and does nothing for the others. us of
// a kernel with one more / so, bf16 means: G = 8, 8 x 10240 pages from 3 tenths of the longest on 22.4 / 19.9, 8 x 4551 from half on 13.6 / 12.0; of a step: G = 4, 2 heads,
// 16 x 22186 37.8 / 36.4, G = 2 56 x 1733 55.8 / 54.5; 20 x 4000 from half on, G = 8, is better with it, 22.9 / 23.9.
inline int score_held_lds(int elem_bytes, int head_dim, int group) {
  constexpr int kLds = 160 << 10;
  const int most = elem_bytes == 2 && head_dim == 64 ? (group == 8 ? 4 : (group == 4 ? 5 : (group == 2 ? 6 : 7))) : 0;
  return most > 0 ? kLds / (most + 1) + 1024 : 0;
}

// Batches of unlike lengths are cut by the lengths on the device: every workgroup finds for itself how many pages each one takes, so
// that the chunks of all sequences together fill kCutSlots workgroups, or a multiple where a chunk would be more than a workgroup can
// hold, and which of them are its own. A chunk is a number of units of 8 pages (whole entries of the group maxima); whole numbers
// but for one quotient (constexpr functions are compiled for the device, too).
// Tiles of a fixed size leave a launch with many workgroups that have no pages, in whose slots those that have some wait, and with
// full tiles that meet on a few units. Two workgroups per compute unit: three or four are no faster but for rows of 128 bytes below
// 96 MB (16 x 128 to 4096 pages, bf16 means, log-uniform lengths 13.1 / 13.8 / 13.5 us; 8 heads, G = 8 on fp32 means have no room for them).
constexpr int kCutSlots = 512;
constexpr int kCutUnit = 8;             // pages
constexpr int kCutMaxBatch = 256;       // four sequences per lane
constexpr int kCutMaxPages = 1 << 20;   // of a sequence
constexpr int kCutMaxUnits = 1 << 22;   // of a launch

// Workgroups for so many units: kCutSlots, or a multiple if chunks of most_units would be more with the sequences' last ones, which are
// the only ones that are not full. `reserve` of them are left to others, which are to run at the same time. three_fit: three to a unit come before four
// (score_cut_three_fit).
constexpr int score_cut_slots(int units, int batch, int most_units, bool three_fit, int reserve) {
  const int need = (units + most_units - 1) / most_units + batch + reserve;
  if (three_fit && need > kCutSlots && need <= kCutSlots * 3 / 2) return kCutSlots * 3 / 2 - reserve;
  return (need + kCutSlots - 1) / kCutSlots * kCutSlots - reserve;
}
// Eight heads on bf16 means. us with four to a unit / three, lengths from 85 hundredths of the longest: 64 x 2000 pages 52.8 / 49.0, 63 x 2951 70.4 / 68;
// from 6 tenths 8 x 27105 72.4 / 69.5. Three where two are enough lose: 16 x 2108 log-uniform 21.3 / 22.8 (a step), 20 x 7000 44.1 / 47.4.
// On fp32 caches only two of them fit, and 768 workgroups are better than 1024 for many sequences all the same: a step of 64 x 4000 pages of one head, log-uniform
// from a quarter of the longest 32.1 / 31.0, 64 x 2200 of 4 from 85 hundredths on 61.1 / 57.8, 64 x 2700 66.6 / 63.1, but 8 x 27105 from 6 tenths on 62.5 / 63.2, 8 x 20000 56.5 / 58.3.
constexpr bool score_cut_three_fit(int group, int head_dim, bool bf16_means, int elem_bytes, int batch) {
  return group == 8 && head_dim == 128 && bf16_means && (elem_bytes == 2 || batch >= 64);
}
// Whether no third workgroup finds a place on a unit.
constexpr bool score_cut_two_fit(int group, int head_dim, bool bf16_means) { return group == 8 && head_dim == 128 && !bf16_means; }
// Units of a chunk at most, so that there are no more than `slots` chunks if the sequences' last ones waste no more than `waste` chunks
// together; with waste = batch that is certain.
constexpr int score_cut_chunk(int units, int slots, int waste, int most_units) {
  const int chunks = slots - waste;
  return units > 0 ? std::min((units + chunks - 1) / chunks, most_units) : 1;
}
// Chunks of a sequence; per_unit: 1 / chunk, off by a few units in the last place at most. The quotient is half a unit or more away
// from the next whole number and off by less for kCutMaxPages. The same function says how many units each of them has, with the chunks in the
// place of the units of one: a sequence's chunks are alike, as full ones and a rest leave a batch of equal lengths uneven (200 x 372 pages 60.8 /
// 54.4 us, 256 x 145 31.7 / 29.4, bf16 means 64 x 752 21.3 / 20.3).
constexpr int score_cut_chunks(int units, int chunk, float per_unit) { return (int)(((float)(units + chunk - 1) + 0.5f) * per_unit); }
// Workgroups that a launch may need, whatever the lengths are.
inline int score_cut_grid(int batch, int max_pages, int most_pages, bool three_fit, int reserve) {
  const int64_t units = (int64_t)batch * ((max_pages + kCutUnit - 1) / kCutUnit);
  return (int)std::min<int64_t>(units, score_cut_slots((int)units, batch, most_pages / kCutUnit, three_fit, reserve));
}

// It costs a round trip for the lengths before that for the page ids and the queries, 0.4 to 0.7 us, 0.2 more above 64 sequences; so
// launches that can be no larger than what is read in a few of these keep their fixed tiles, and so do batches known to be nearly even,
// whose tiles are large. kernel us with fixed tiles / so (8 heads, G = 4, D = 128 unless it says otherwise; lengths log-uniform from a
// 30th, or uniform from a tenth of the longest; nothing in the caches):
//   fp32 means, 16 x 4096 pages log 23.3 / 20.3, uniform 28.8 / 26.8; 32 x 2048 21.3 / 15.9, 30.0 / 26.0; 64 x 1024 28.9 / 15.0, 32.9 / 26.4;
//   80 x 1000 36.2 / 19.2; 256 x 1024 102 / 63; 4 x 32768 42.3 / 41.7, 61.3 / 58.9; G = 8 32 x 2048 27.6 / 17.2, 37.0 / 27.5
//   bf16 means, 16 x 4096 14.5 / 13.0; 64 x 1024 18.2 / 10.5; 12 x 3125 uniform 15.2 / 12.5
//   one of 16 x 8192 pages, the others a quarter as long: fp32 means 40.5 / 28.5, bf16 means 22.9 / 16.9
// By the bytes of the longest sequence times the batch, log / uniform: 32 MB 3 sequences 6.2 / 6.4, 6.6 / 6.9, 16 6.2 / 5.9, 7.0 / 7.3; 48 MB 3 x
// 8.3 / 8.0, 16 x 8.1 / 7.4, 8.6 / 8.1; 64 MB 6 x 32 heads, G = 1, 7.7 / 7.8, 10.4 / 10.9, 16 x 11.0 / 6.7, 13.8 / 9.9; rows of 128 bytes (D = 64,
// bf16 means) at 64 MB 16 x 7.8 / 7.2, 9.9 / 10.3, 100 x 10.5 / 11.9, at 128 MB 12.9 / 12.2, 17.8 / 17.9 and 11.7 / 10.8, 16.4 / 16.7.
// Lengths within a factor of two, uniform: from 6.5 tenths of the longest at 100 MB 17.2 / 17.7, at 130 MB 24 x 22.2 / 22.5, at 145 MB 24 x 28.2 /
// 22.9, at 300 MB 50.5 / 42.9; from 8 tenths at 400 MB 12 x 66.2 / 62.9; from 9 tenths at 180 MB 60 x 0.98 times as fast; 4 sequences of 16 heads, G
// = 1, D = 64 at 400 MB 0.94 times. With every other sequence just half as long it is even at best (16 x 8192 64.8 / 65.8, bf16 means 35.5 /
// 36.5), and so it is for two sequences (2 x 16384 uniform 20.4 / 20.5).
// Above 64 sequences, four to a lane, the way to a chunk is longer and what short sequences are cut into coarse: 128 x 12 to 96 pages 8.8 / 9.2, from 7
// tenths on 12.4 / 12.9, even 256 x 96 19.6 / 20.6; 100 x 12 to 240 log 10.2 / 6.5, 128 x 20 to 188 uniform 16.5 / 14.4.
// Without a lower bound (min_pages = 0) a batch may be even and gain nothing, so what even ones do not lose decides, a narrow range of lengths as little:
// fp32 means, even 64 x 248 pages (63 MB) 15.8 / 16.7, 16 x 868 14.9 / 15.2, but 71 MB 4 x 19.1 / 17.6, 16 x 19.1 / 17.6, 64 x 19.3 / 17.7, 100 MB 64 x 22.2 / 20.1, 150 MB
// 16 x 28.1 / 28.2, 300 MB 53.3 / 51.3; bf16 means, 50 MB 64 x 13.5 / 14.1, but 55 MB 16 x 17.4 / 14.9, 64 x 17.4 / 15.5, 150 MB 64 x 30.0 / 28.2; above 64
// sequences 50 MB 65 x 13.2 / 13.9, 128 x 193 from 7 tenths on (85 MB) 18.2 / 19.0, but 99 MB even 128 x 22.0 / 20.8, 200 x 21.9 / 21.2, 149 MB 128 x 29.4 / 28.8, 200 x 29.0 /
// 29.7, 219 MB 140 x 42.6 / 41.3, log-uniform 128 x 193 13.6 / 10.8.
inline bool score_cuts(int batch, int max_pages, int min_pages, int mean_bytes, int64_t rec_bytes) {
  if (batch < 3 || batch > kCutMaxBatch || max_pages > kCutMaxPages) return false;
  if ((int64_t)batch * ((max_pages + kCutUnit - 1) / kCutUnit) > kCutMaxUnits) return false;
  const int64_t most = (int64_t)batch * max_pages * rec_bytes;
  if (min_pages >= (max_pages + 1) / 2) return batch >= 8 && mean_bytes > 128 && min_pages <= max_pages / 8 * 7 && most >= (144ll << 20);
  if (batch > 64 && max_pages < 128) return false;
  if (batch < 16 || mean_bytes <= 128 || (batch > 64 && min_pages == 0)) return most >= (96ll << 20);
  return most >= ((min_pages > 0 ? 48ll : (mean_bytes > 256 ? 68ll : 52ll)) << 20);
}

// A decode step renews the statistics of the page that has received a token before that page is scored: in the workgroup whose tile it is in,
// which takes two more round trips and some hundred instructions, or in workgroups of its own, a KV head to a wave, which come first or last
// in the grid.
enum LastPage { kLastPageNone, kLastPageInTile = 1, kLastPageOwn = 2, kLastPageFirst = 4, kLastPageBits = 3 };
constexpr int last_page_groups(int kv_heads) { return (kv_heads + 3) / 4; }

// Workgroups of their own cost the units that they land on what they read, and on these units a launch that gives every unit the same ends
// later; a small launch, which is a chain of latencies, gains by them, and so do large ones, in which a late start of some tiles shows.
// In launches of at most one workgroup per unit they are best first; in larger ones they then leave some units one more than others (16 x 8192 pages
// 141.3 in the tile, 157.3 first, 140.4 last). Between 44 and 192 MB the bytes decide, from batches of 16 and 24 sequences; one or two long
// ones there were measured with a fitted tile only.
// A step us in the tile / so (8 heads, G = 4, D = 128): fp32 means, 1 x 1000 pages 16.2 / 14.5, 1 x 2048 18.2 / 16.6, 2 x 3000 20.8 / 19.3, 16 x 400
// 20.3 / 18.1, bf16 means, pages of 8, 4 x 4096 23.6 / 20.9, 32 x 600 21.6 / 19.7; but fp32 means 16 x 1000 (67 MB) 31.3 / 32.5, 24 x 1000 44.9 / 45.6,
// bf16 means 24 x 1000 (52 MB) 23.8 / 25.8; large: 4 x 16384 65.3 / 64.8, 80 x 4096, pages of 8 157.2 / 155.7, 48 x 2048 bf16 means 121.4 / 119.5, 160 x 700 fp32
// means (320 of them) 183.3 / 184.3. Cut by the lengths: 32 x 4K-131K tokens 64.8 / 64.4, 16 x 1000 29.2 / 28.3, bf16 means 20.3 / 18.3. With 8 query
// heads two workgroups fill a unit and the last ones wait for a place: 3 x 20000 pages of 32, cut, 60.5 / 63.1, but 24 x 1000 61.5 / 58.7.
// A tile that was fitted to an even batch (`fitted`) leaves the last workgroup of a sequence about as many pages as the others, and renewing one of them
// comes on top: a step with the tile of score_tile / fitted, in the tile / fitted, last: 78 x 142 pages of 16 heads, bf16 means (45 MB), 66.0 / 67.4 / 63.3, 2 x 13697
// 40.0 / 41.6 / 39.6, 60 x 588 of 16 heads 117.8 / 116.3 / 113.3, 10 x 2578 28.7 / 29.0 / 27.6, fp32 means 7 x 1161 of 16 heads 33.1 / 30.6 / 29.9; 120 x 810 of D = 64
// 54.3 / 52.4 / 52.7.
inline int score_last_page_rule(bool cut, int64_t workgroups, int last_pages, int64_t bytes, int group, bool fitted = false) {
  constexpr int kNumCUs = 256;
  if (cut) return group == 8 && bytes > (128ll << 20) ? kLastPageInTile : kLastPageOwn;
  if (bytes <= (44ll << 20)) return workgroups <= kNumCUs ? (kLastPageOwn | kLastPageFirst) : kLastPageOwn;
  return group < 8 && last_pages <= (fitted ? 2 * kNumCUs : (bytes >= (192ll << 20) ? kNumCUs : 0)) ? kLastPageOwn : kLastPageInTile;
}

// Workgroups that a cut leaves to last pages, so that they run with the chunks where no third finds a place on a unit.
inline int score_cut_reserve(bool refresh_tail, int batch, int kv_heads, int64_t bytes, int group, bool two_fit) {
  const int last_pages = last_page_groups(kv_heads) * batch;
  return two_fit && refresh_tail && (score_last_page_rule(true, 0, last_pages, bytes, group) & kLastPageOwn) ? last_pages : 0;
}

// The grid of a launch with `tiles` tiles to a sequence, or to the batch where it is cut by its lengths, and its `refresh` argument: a LastPage and,
// above its bits, the rows of the grid that are for last pages, or the first workgroup that is. fitted: the tile is score_even_tile's own.
struct ScoreGrid {
  int x, y, refresh;
};
constexpr int kMaxGridRows = 65535;
inline ScoreGrid score_grid(bool cut, int tiles, int batch, int kv_heads, bool refresh_tail, int64_t bytes, int group, bool fitted) {
  const int last_pages = last_page_groups(kv_heads) * batch;
  ScoreGrid g = {tiles, cut ? 1 : batch, kLastPageNone};
  if (refresh_tail) g.refresh = score_last_page_rule(cut, (int64_t)g.x * g.y, last_pages, bytes, group, fitted);
  if (!(g.refresh & kLastPageOwn)) return g;
  const int rows = (last_pages + tiles - 1) / tiles;
  if (!cut && batch + rows > kMaxGridRows) {  // more sequences than a launch could have rows for beside them, of a few pages each
    g.refresh = kLastPageInTile;
    return g;
  }
  g.refresh |= (cut ? tiles : rows) << kLastPageBits;
  if (cut) g.x += last_pages;
  else g.y += rows;
  return g;
}

}  // namespace unique
