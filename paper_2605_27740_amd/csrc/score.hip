// Fused page-score kernel (Eq. 6 of the paper; Eq. 3 when G = 1):
//   score(p) = max_g [ q_g . mean_p + lambda * |q_g|_2 * std_p ]   per (sequence, KV head, logical page).
// The G x P intermediate never exists in memory: the G dot products, the rank-one offset and the max
// over the group are all formed in registers and one float per (KV head, page) is written.
//
// Layout of the work: 8 lanes own one (page, KV head) mean row and read it as 16-byte chunks (D/32
// of them for fp32 means, D/64 for bf16 means) each, so a wave covers 8 consecutive head rows per step -- with 8 KV heads that is exactly one
// page record, read as one contiguous block whatever the page table does to page placement, with
// the page's stds taken from the tail of the same record. Every lane keeps its slices of the G
// queries of its (fixed) KV head in registers for the whole kernel. The G partial dot products are
// reduced over the 8 lanes with three DPP steps. The page-table entries of all of a wave's steps are
// fetched up front (together with the sequence length and the queries, so the prologue is two memory
// round trips); two or four records are in flight per wave, requested with unconditional loads so that the
// loop is straight-line code with exact waits. Scores of a tile are staged in LDS and written as one
// contiguous run per KV head (4-byte scattered stores cost a tenth of the kernel otherwise).
#include <type_traits>

#include "score_core.hpp"
#include "score_tile.hpp"

namespace unique {
namespace {

constexpr int kScoreWaves = 4;

// Statistics of the last (possibly partial) page of sequence b, recomputed from the keys by the whole
// workgroup: wave w takes KV heads w, w+4, ... The page size is a run-time value here.
template <typename T, int D>
__device__ __forceinline__ void refresh_tail_record(const CacheView& c, int b, int N, int P) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;  // wave: scalar
  const int p = P - 1, S = c.S;
  const int n = min(S, N - p * S);
  const int64_t phys = c.page_table[(int64_t)b * c.max_pages + p];
  if (phys < 0 || phys >= c.num_phys || n < 1) return;
  char* rec = reinterpret_cast<char*>(c.page_stats) + phys * c.rec_bytes;
  const int elem = c.stats_bf16 ? 2 : 4;
  for (int hkv = wave; hkv < c.Hkv; hkv += kScoreWaves) {
    PageRefresh<T, D, 32> page;  // page_size <= 32
    page.request(reinterpret_cast<const T*>(c.k_cache) + phys * c.kv_page_stride + hkv * c.kv_head_stride, n, lane);
    page.reduce(n, lane);
    page.store_mean(rec + (int64_t)hkv * D * elem, c.stats_bf16, lane);
    if (lane == 0) reinterpret_cast<float*>(rec + (int64_t)c.Hkv * D * elem)[hkv] = page.std;
  }
}

// The last (possibly partial) page of sequence b for KV head h, by one wave: its statistics are recomputed from its keys and stored, and it is
// scored with them, from `mean`, D elements of LDS. The page size is a run-time value here.
template <typename T, typename TS, int D, int G, int kMaxTokens>
__device__ __forceinline__ void refresh_and_score(const CacheView& c, RowScorer<T, TS, D, G>& scorer, float lambda, int phys, int n, int h,
                                                  TS* mean, float* score) {
  using Scorer = RowScorer<T, TS, D, G>;
  const int lane = threadIdx.x % kWave;
  PageRefresh<T, D, kMaxTokens> page;
  page.request(reinterpret_cast<const T*>(c.k_cache) + (int64_t)phys * c.kv_page_stride + (int64_t)h * c.kv_head_stride, n, lane);
  page.reduce(n, lane);
  page.store_mean(mean, sizeof(TS) == 2, lane);
  char* rec = reinterpret_cast<char*>(c.page_stats) + (int64_t)phys * c.rec_bytes;
  page.store_mean(rec + (int64_t)h * D * (int)sizeof(TS), sizeof(TS) == 2, lane);
  if (lane == 0) reinterpret_cast<float*>(rec + (int64_t)c.Hkv * D * (int)sizeof(TS))[h] = page.std;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_sched_barrier(0);  // (unpacked earlier the queries would take the registers of two more waves)
  scorer.unpack(lambda);
  Raw16 md[Scorer::kChunks];
#pragma unroll
  for (int j = 0; j < Scorer::kChunks; ++j) md[j] = load_raw(mean + lane % kRowLanes * Scorer::kE + j * (Scorer::kE * kRowLanes));
  const float s = scorer.score(md, page.std);
  if (lane == 0) *score = s;
}
template <typename T, typename TS, int D, int G>
__device__ __forceinline__ void score_last_page(const CacheView& c, const T* q, float lambda, int b, int h, TS* mean, int score_stride,
                                                float* scores) {
  const int lane = threadIdx.x % kWave;
  const int32_t* pt = c.page_table + (int64_t)b * c.max_pages;
  // the last of the page ids that there may be are requested with the length, and most often the last page's is one of them
  const int late = pt[max(c.max_pages_hint - 1 - lane, 0)];
  const int N = c.seq_lens[b];
  RowScorer<T, TS, D, G> scorer;
  scorer.request(q + ((int64_t)b * c.H + h * G) * D, lane % kRowLanes);
  const int P = min((N + c.S - 1) / c.S, c.max_pages_hint);
  if (P < 1) return;
  const int phys = __builtin_amdgcn_readfirstlane(c.max_pages_hint - P < kWave ? __builtin_amdgcn_readlane(late, c.max_pages_hint - P) : pt[P - 1]);
  float* score = scores + ((int64_t)b * c.Hkv + h) * score_stride + P - 1;
  if (phys < 0 || (int64_t)phys >= c.num_phys) {
    if (lane == 0) *score = __uint_as_float(0x7fc00000u);  // as below
    return;
  }
  const int n = min(c.S, N - (P - 1) * c.S);
  if (c.S == 8) refresh_and_score<T, TS, D, G, 8>(c, scorer, lambda, phys, n, h, mean, score);
  else if (c.S == 16) refresh_and_score<T, TS, D, G, 16>(c, scorer, lambda, phys, n, h, mean, score);
  else refresh_and_score<T, TS, D, G, 32>(c, scorer, lambda, phys, n, h, mean, score);
}

// The chunk of this workgroup, pages [first, first + pages) of sequence b or fewer, where the batch is cut by its lengths (score_tile.hpp);
// N: the sequence's length, P: its pages without the last `less`. w: the workgroup. false: there are no more chunks. most_pages: of a chunk;
// three_fit, reserve: see score_cut_slots. kSeqs: consecutive sequences that a lane looks after (four for every batch cost 64 or fewer 0.3 us).
template <int kSeqs>
__device__ __forceinline__ bool find_chunk(const CacheView& c, int w, int most_pages, bool three_fit, int reserve, int less, int& b, int& first, int& pages,
                                           int& N, int& P) {
  const int lane = threadIdx.x % kWave;
  const int page_shift = __ffs(c.S) - 1;  // page sizes are powers of two
  int len[kSeqs], units[kSeqs], all = 0;
#pragma unroll
  for (int i = 0; i < kSeqs; ++i) len[i] = lane * kSeqs + i < c.B ? c.seq_lens[lane * kSeqs + i] : 0;
#pragma unroll
  for (int i = 0; i < kSeqs; ++i) {
    const int n = max(0, min((len[i] + c.S - 1) >> page_shift, c.max_pages_hint) - less);
    units[i] = (n + kCutUnit - 1) / kCutUnit;
    all += units[i];
  }
  all = __builtin_amdgcn_readlane(wave_inclusive_scan(all), kWave - 1);
  const int most = most_pages / kCutUnit, slots = score_cut_slots(all, c.B, most, three_fit, reserve);
  int chunk, chunks[kSeqs], mine, upto;
  auto cut = [&](int waste) {
    chunk = score_cut_chunk(all, slots, waste, most);
    const float per_unit = __builtin_amdgcn_rcpf((float)chunk);
    mine = 0;
#pragma unroll
    for (int i = 0; i < kSeqs; ++i) {
      chunks[i] = score_cut_chunks(units[i], chunk, per_unit);
      mine += chunks[i];
    }
    upto = wave_inclusive_scan(mine);
  };
  cut(c.B / 2);
  if (__builtin_amdgcn_readlane(upto, kWave - 1) > slots) cut(c.B);  // uniform
  const unsigned long long behind = __ballot(upto > w);
  if (behind == 0) return false;
  const int at = __ffsll(behind) - 1;
  int i = w - __builtin_amdgcn_readlane(upto - mine, at), s = 0, n = __builtin_amdgcn_readlane(len[0], at), parts = __builtin_amdgcn_readlane(chunks[0], at);
#pragma unroll
  for (int j = 1; j < kSeqs; ++j) {
    const int next = __builtin_amdgcn_readlane(len[j], at), next_parts = __builtin_amdgcn_readlane(chunks[j], at);
    const bool on = s == j - 1 && i >= parts;
    i -= on ? parts : 0;
    s = on ? j : s;
    n = on ? next : n;
    parts = on ? next_parts : parts;
  }
  b = at * kSeqs + s;
  N = n;
  P = min((N + c.S - 1) >> page_shift, c.max_pages_hint) - less;
  pages = score_cut_chunks((P + kCutUnit - 1) / kCutUnit, parts, __builtin_amdgcn_rcpf((float)parts)) * kCutUnit;
  first = i * pages;
  return true;
}

// T: element type of q; TS: element type of the stored means (float, or bf16_t for bf16 statistics). The arguments are in an order
// without gaps: 8 bytes more cost a small launch 0.2 us (16 x 400 pages 7.5 / 7.3).
// kNT: the records are read with non-temporal loads (a launch that streams more than the caches hold).
// refresh: who renews the last page of every sequence before it is scored, a LastPage, and above its bits where these workgroups are (the grid's
// extent would have to be fetched).
// kOwn: last pages have workgroups of their own. (Where they have not, their code in the kernel would cost 0.3 to 0.8 us.)
// kCut: 0: grid (tile, sequence), tile_pages to each; else the batch is cut by its lengths (find_chunk), tile_pages at most to a chunk.
template <typename T, typename TS, int D, int G, bool kNT, int kCut, bool kOwn>
__global__ __launch_bounds__(kScoreWaves* kWave) void page_score_kernel(CacheView c, const T* __restrict__ q, float lambda, int score_stride,
                                                                        float* __restrict__ scores, float* __restrict__ scores_out,
                                                                        uint32_t* __restrict__ group_max, int refresh,
                                                                        int tile_pages) {
  using Scorer = RowScorer<T, TS, D, G>;
  constexpr int kE = Scorer::kE, kChunks = Scorer::kChunks;
  // Records in flight per wave. bf16 means in launches that stream from memory: four (80 x 4096 pages 117 us, two 122);
  // with fp32 means, twice the bytes, four records are no faster (16 x 8192 pages 87 us, two 86) and cost small launches
  // 1 us (2048 pages 8.0, two 7.0).
  constexpr int kDepth = sizeof(TS) == 2 && kNT ? 4 : 2;

  extern __shared__ __attribute__((aligned(16))) float tile_scores[];  // [Hkv][tile_stride]
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;  // wave: scalar
  constexpr int less = kOwn;  // pages that this workgroup's sequence has elsewhere
  int row = blockIdx.y;       // of the grid; those beyond the sequences are for last pages
  if constexpr (kOwn) {
    const int groups = last_page_groups(c.Hkv), extra = refresh >> kLastPageBits;  // rows of them, or the workgroup that is the first
    if (kCut == 0 && (refresh & kLastPageFirst)) row = row < extra ? c.B + row : row - extra;
    const int at = kCut > 0 ? (int)blockIdx.x - extra : (row < c.B ? -1 : (int)blockIdx.x * extra + row - c.B);
    if (at >= 0) {
      const int which = at / groups, h = at % groups * kScoreWaves + wave;
      if (which < c.B && h < c.Hkv)
        score_last_page<T, TS, D, G>(c, q, lambda, which, h, reinterpret_cast<TS*>(tile_scores) + wave * D, score_stride, scores);
      return;
    }
  }
  int b, tile0, N, P;
  if constexpr (kCut > 0) {
    const bool three_fit = score_cut_three_fit(G, D, sizeof(TS) == 2, sizeof(T), c.B);
    const int reserve = kOwn && score_cut_two_fit(G, D, sizeof(TS) == 2) ? last_page_groups(c.Hkv) * c.B : 0;
    if (!find_chunk<kCut>(c, blockIdx.x, tile_pages, three_fit, reserve, less, b, tile0, tile_pages, N, P)) return;
  } else {
    b = row;
    tile0 = blockIdx.x * tile_pages;  // tile_pages logical pages per workgroup (a multiple of 8, up to 256)
  }
  const int tshift = 32 - __clz(tile_pages - 1), tile_stride = 1 << tshift;  // score_tile_stride
  const int row8 = lane / kRowLanes, cl = lane % kRowLanes;
  // which head and which page of a step this lane's row is; both fixed for the whole kernel
  int hkv, page_in_step, pages_per_step, wave_slot, wave_slots;
  if (c.Hkv >= kRowsPerWave) {
    const int slots_per_page = c.Hkv / kRowsPerWave;  // a page record spans this many wave steps
    hkv = (wave % slots_per_page) * kRowsPerWave + row8;
    page_in_step = 0;
    pages_per_step = 1;
    wave_slot = wave / slots_per_page;
    wave_slots = kScoreWaves / slots_per_page;
  } else {
    pages_per_step = kRowsPerWave / c.Hkv;
    hkv = row8 % c.Hkv;
    page_in_step = row8 / c.Hkv;
    wave_slot = wave;
    wave_slots = kScoreWaves;
  }
  const int step_pages = wave_slots * pages_per_step;  // pages the workgroup advances per step

  // A tile that may lie beyond its sequence looks at the length before it asks for anything else: in a ragged batch most
  // workgroups are such tiles, and each kept a slot for the two round trips below (32 x 128 to 4096 pages 22.2 -> 21.8 us).
  // Without a known bound every tile would look first, which costs an even batch 3 % (16 x 8192 pages of one head 40.6 ->
  // 41.9).
  if (kCut == 0 && c.min_pages_hint > 0 && tile0 >= c.min_pages_hint && tile0 >= (c.seq_lens[b] + c.S - 1) / c.S - less) return;

  // The sequence length, the page ids of all of this wave's steps (lane L holds entry L = step *
  // pages_per_step + page_in_step) and the queries are requested together; the page-table row always has
  // max_pages readable entries, so its load does not have to wait for the page count.
  const int32_t* pt = c.page_table + (int64_t)b * c.max_pages;
  int my_page, my_phys_raw = -1;
  {
    const int st = lane / pages_per_step, po = lane % pages_per_step;
    my_page = tile0 + (wave_slot + st * wave_slots) * pages_per_step + po;
    if (my_page < min(tile0 + tile_pages, kCut > 0 ? P : c.max_pages_hint)) my_phys_raw = pt[my_page];
  }
  if constexpr (kCut == 0) N = c.seq_lens[b];
  Scorer scorer;
  scorer.request(q + ((int64_t)b * c.H + hkv * G) * D, cl);
  if constexpr (kCut == 0) {
    P = min((N + c.S - 1) / c.S, c.max_pages_hint) - less;  // pages beyond the host bound are ignored
    if (tile0 >= P) return;
  }
  const int tile_end = min(tile0 + tile_pages, P);
  if (!kOwn && refresh && tile_end == P) {  // this workgroup scores the last page: bring its record up to date first
    refresh_tail_record<T, D>(c, b, N, P);
    __threadfence_block();
    __syncthreads();
  }

  const char* stats = reinterpret_cast<const char*>(c.page_stats);
  const int64_t std_off = (int64_t)c.Hkv * D * (int64_t)sizeof(TS);  // byte offset of the stds inside a record

  const int n_steps = (tile_end - (tile0 + wave_slot * pages_per_step) + step_pages - 1) / step_pages;  // may be <= 0
  const int my_phys = (my_page < tile_end && my_phys_raw >= 0 && (int64_t)my_phys_raw < c.num_phys) ? my_phys_raw : -1;

  // A ring of kDepth records is in flight per wave. The loads are unconditional -- a step past the end
  // of the tile, or one whose page id is invalid, reads the first bytes of the statistics instead, which
  // costs no memory traffic -- so the loop is straight-line code and every wait names the exact number of
  // requests that may stay outstanding.
  Raw16 ring[kDepth][kChunks];
  float ring_sd[kDepth];
  int ring_phys[kDepth];
  auto issue = [&](int st, Raw16(&md)[kChunks], float& sd, int& phys) {
    const int src_lane = min(st * pages_per_step + page_in_step, kWave - 1);
    const int ph = pages_per_step == 1 ? __builtin_amdgcn_readlane(my_phys, min(st, kWave - 1))
                                       : __shfl(my_phys, src_lane, kWave);
    phys = st < n_steps ? ph : -1;
    const char* rec = stats + (int64_t)max(phys, 0) * c.rec_bytes;
    const TS* row = phys >= 0 ? reinterpret_cast<const TS*>(rec) + hkv * D + cl * kE : reinterpret_cast<const TS*>(stats);
#pragma unroll
    for (int j = 0; j < kChunks; ++j) md[j] = load_raw_stream(row + j * (kE * kRowLanes), kNT);
    sd = reinterpret_cast<const float*>(rec + std_off)[hkv];
  };
  auto consume = [&](int st, const Raw16(&mc)[kChunks], float sd_cur, int phys_cur) {
    const float best = scorer.score(mc, sd_cur);
    const int p = tile0 + (wave_slot + st * wave_slots) * pages_per_step + page_in_step;
    // a page whose table entry points outside the pool gets NaN, which ranks below every score
    if (cl == 0 && p < tile_end) tile_scores[hkv * tile_stride + p - tile0] = phys_cur >= 0 ? best : __uint_as_float(0x7fc00000u);
  };
#pragma unroll
  for (int u = 0; u < kDepth; ++u) issue(u, ring[u], ring_sd[u], ring_phys[u]);
  scorer.unpack(lambda);  // the queries arrived with the page ids; they are unpacked while the first records are on their way
  for (int st0 = 0; st0 < n_steps; st0 += kDepth) {
#pragma unroll
    for (int u = 0; u < kDepth; ++u) {
      consume(st0 + u, ring[u], ring_sd[u], ring_phys[u]);
      issue(st0 + u + kDepth, ring[u], ring_sd[u], ring_phys[u]);
    }
  }
  __syncthreads();
  // the tile's scores leave as one contiguous run per KV head
  const int tile_len = tile_end - tile0;
  for (int idx = threadIdx.x; idx < c.Hkv * tile_stride; idx += kScoreWaves * kWave) {
    const int h = idx >> tshift, pp = idx & (tile_stride - 1);
    if (pp < tile_len) {
      const float v = tile_scores[idx];
      scores[((int64_t)b * c.Hkv + h) * score_stride + tile0 + pp] = v;
      if (scores_out) scores_out[((int64_t)b * c.Hkv + h) * c.max_pages + tile0 + pp] = v;
    }
  }
  if (group_max) {  // a thread per group of pages; tiles are multiples of it
    for (int idx = threadIdx.x; idx < c.Hkv * tile_stride / kGroupPages; idx += kScoreWaves * kWave) {
      const int first = idx * kGroupPages, h = first >> tshift, pp = first & (tile_stride - 1);
      if (pp >= tile_len) continue;
      float top = __uint_as_float(0x7fc00000u);  // the maximum ignores NaN
#pragma unroll
      for (int i = 0; i < kGroupPages; i += 4) {
        const float4 v = *reinterpret_cast<const float4*>(&tile_scores[first + i]);
        top = fmaxf(top, v.x);
        top = pp + i + 1 < tile_len ? fmaxf(top, v.y) : top;
        top = pp + i + 2 < tile_len ? fmaxf(top, v.z) : top;
        top = pp + i + 3 < tile_len ? fmaxf(top, v.w) : top;
        if (pp + i + 4 >= tile_len) break;
      }
      group_max[((int64_t)b * c.Hkv + h) * (score_stride / kGroupPages) + (tile0 + pp) / kGroupPages] = score_key(top);
    }
  }
}

template <typename T, int D, int G>
hipError_t launch_t(const CacheView& cv, const void* q, float lambda, float* scores, int stride, float* out,
                    uint32_t* group_max, bool refresh_tail, hipStream_t st) {
  const CacheView& c = cv;
  const bool nt = (int64_t)c.B * c.max_pages_hint * c.rec_bytes > kStreamNtBytes;
  // A wave keeps the page ids of all its steps in its 64 lanes, which caps the tile at 64 pages per wave
  // slot (4 slots up to 8 KV heads, 2 at 16, 1 when one wave steps through all 32 heads of a page alone).
  const int wave_slots = c.Hkv <= 8 ? kScoreWaves : kScoreWaves * kRowsPerWave / c.Hkv;
  const int mean_bytes = D * (c.stats_bf16 ? 2 : 4), most = 64 * wave_slots;
  const bool cut = score_cuts(c.B, c.max_pages_hint, c.min_pages_hint, mean_bytes, c.rec_bytes);
  const int plain = cut ? most : score_tile(c.B, c.Hkv, D, c.max_pages_hint, c.min_pages_hint, most);
  const int tile = cut ? most : score_even_tile(plain, c.B, c.max_pages_hint, c.min_pages_hint, mean_bytes, most);
  const int64_t bytes = (int64_t)c.B * c.max_pages_hint * c.rec_bytes;
  const int reserve = score_cut_reserve(refresh_tail, c.B, c.Hkv, bytes, G, score_cut_two_fit(G, D, c.stats_bf16));
  const int tiles = cut ? score_cut_grid(c.B, c.max_pages_hint, tile, score_cut_three_fit(G, D, c.stats_bf16, (int)sizeof(T), c.B), reserve)
                        : (c.max_pages_hint + tile - 1) / tile;
  const ScoreGrid grid = score_grid(cut, tiles, c.B, c.Hkv, refresh_tail, bytes, G, tile != plain);
  const int refresh = grid.refresh;
  size_t lds = (size_t)c.Hkv * score_tile_stride(tile) * sizeof(float);
  if (refresh & kLastPageOwn) lds = std::max<size_t>(lds, kScoreWaves * mean_bytes);
  if (!cut) lds = (size_t)std::max(score_lds((int)lds, (int)sizeof(T), D, G, (int64_t)tiles * c.B), score_held_lds((int)sizeof(T), D, G));
  auto go = [&](auto kernel) {
    kernel<<<dim3(grid.x, grid.y), dim3(kScoreWaves * kWave), lds, st>>>(c, reinterpret_cast<const T*>(q), lambda, stride, scores, out, group_max,
                                                         refresh, tile);
    return hipGetLastError();
  };
  auto with = [&](auto mean, auto stream_nt) {
    using TS = decltype(mean);
    constexpr bool kNT = decltype(stream_nt)::value;
    auto of = [&](auto seqs) {
      constexpr int kCut = decltype(seqs)::value;
      return refresh & kLastPageOwn ? go(page_score_kernel<T, TS, D, G, kNT, kCut, true>) : go(page_score_kernel<T, TS, D, G, kNT, kCut, false>);
    };
    if (!cut) return of(std::integral_constant<int, 0>());
    return c.B <= kWave ? of(std::integral_constant<int, 1>()) : of(std::integral_constant<int, kCutMaxBatch / kWave>());
  };
  if (c.stats_bf16) return nt ? with(bf16_t(), std::true_type()) : with(bf16_t(), std::false_type());
  return nt ? with(float(), std::true_type()) : with(float(), std::false_type());
}

template <typename T, int D>
hipError_t dispatch_g(const CacheView& c, const void* q, float lambda, float* scores, int stride, float* out,
                      uint32_t* group_max, bool refresh_tail, hipStream_t st) {
  switch (c.H / c.Hkv) {
    case 1: return launch_t<T, D, 1>(c, q, lambda, scores, stride, out, group_max, refresh_tail, st);
    case 2: return launch_t<T, D, 2>(c, q, lambda, scores, stride, out, group_max, refresh_tail, st);
    case 4: return launch_t<T, D, 4>(c, q, lambda, scores, stride, out, group_max, refresh_tail, st);
    case 8: return launch_t<T, D, 8>(c, q, lambda, scores, stride, out, group_max, refresh_tail, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

bool score_supported(int dtype, int D, int G, int Hkv) {
  if (!(dtype == 0 || dtype == 1) || !(D == 64 || D == 128)) return false;
  if (!(G == 1 || G == 2 || G == 4 || G == 8)) return false;
  // a wave covers 8 head rows per step; the 4 waves of a workgroup must tile whole page records
  return Hkv == 1 || Hkv == 2 || Hkv == 4 || Hkv == 8 || Hkv == 16 || Hkv == 32;
}

hipError_t launch_score(const CacheView& c, const void* d_q, float lambda, float* d_scores, int score_stride,
                        float* d_scores_out, uint32_t* d_group_max, bool refresh_tail, hipStream_t stream) {
  if (refresh_tail && d_scores_out) return hipErrorInvalidValue;  // last pages with workgroups of their own leave no second copy of their score
  if (c.dtype == 0) {
    return c.D == 64 ? dispatch_g<float, 64>(c, d_q, lambda, d_scores, score_stride, d_scores_out, d_group_max, refresh_tail, stream)
                     : dispatch_g<float, 128>(c, d_q, lambda, d_scores, score_stride, d_scores_out, d_group_max, refresh_tail, stream);
  }
  return c.D == 64 ? dispatch_g<bf16_t, 64>(c, d_q, lambda, d_scores, score_stride, d_scores_out, d_group_max, refresh_tail, stream)
                   : dispatch_g<bf16_t, 128>(c, d_q, lambda, d_scores, score_stride, d_scores_out, d_group_max, refresh_tail, stream);
}

}  // namespace unique
