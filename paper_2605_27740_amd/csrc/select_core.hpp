// The selection of the top-k pages of one row by one workgroup, over keys in registers: the device code that the selection
// kernels (select.hip, which explains the search) and the kernels that attend over the selected pages at once (step.hip) share.
#pragma once
#include "device_utils.hpp"
#include "kernels.hpp"

namespace unique {
namespace {

constexpr int kMaxRankCandidates = 512;  // above this the boundary bucket is resolved by radix rounds
constexpr uint32_t kKeyForced = 0xffffffffu;  // key of a page that is selected whatever its score
constexpr uint32_t kKeyNegInf = 0x007fffffu, kKeyPosInf = 0xff800000u;  // keys of -inf and +inf

__device__ __forceinline__ float ordered_to_float(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// Bucket of a key in a histogram of n_buckets buckets that is linear in the score between lo and the row
// maximum (scale = (n_buckets - 1) / range): monotone in the score, so bucket order never contradicts
// score order. -inf and NaN go to the lowest bucket, +inf and always-selected pages to the highest.
__device__ __forceinline__ int linear_bucket(uint32_t k, float lo, float scale, int n_buckets) {
  if (k >= kKeyPosInf) return n_buckets - 1;
  if (k > kKeyNegInf) return min(n_buckets - 1, max(0, (int)((ordered_to_float(k) - lo) * scale)));
  return 0;
}

// Lanes of one wave whose predicate holds and which come before this lane, added to `acc`.
__device__ __forceinline__ int lanes_before(unsigned long long mask, int acc) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, (uint32_t)acc));
}

// hist[bin] += 1 for every active lane, as one addition where they all have the same bin: 64 lanes adding to one address
// take about 800 cycles, and masses of equal keys are what the radix rounds are for.
__device__ __forceinline__ void add_one(int* hist, int bin) {
  const unsigned long long active = __ballot(1);
  if (__all(bin == __builtin_amdgcn_readfirstlane(bin))) {
    if (lanes_before(active, 0) == 0) atomicAdd(&hist[bin], __popcll(active));
  } else {
    atomicAdd(&hist[bin], 1);
  }
}

// One round-set of 8-bit radix selection over the keys accepted by `keep(j)`: returns the exact key of
// the need-th largest accepted key and leaves in `need` how many keys equal to it must be taken.
// hist: 256 ints of LDS; s_prefix / s_need: LDS scalars. All threads of the workgroup must call it.
// kStatic > 0: the per-thread item count is that constant (items live in registers, loops unroll).
template <int kThreads, int kStatic, typename KeyAt, typename Keep>
__device__ __forceinline__ uint32_t radix_threshold(int n_items, KeyAt key_at, Keep keep, int& need, int* hist,
                                                    uint32_t* s_prefix, int* s_need) {
  const int t = threadIdx.x;
  const int n = kStatic > 0 ? kStatic : n_items;
  uint32_t prefix = 0;
#pragma unroll 1
  for (int round = 0; round < 4; ++round) {
    const int shift = 24 - 8 * round;
    __syncthreads();  // everyone is done with the previous contents of hist
    for (int i = t; i < 256; i += kThreads) hist[i] = 0;
    __syncthreads();
    if constexpr (kStatic > 0) {
#pragma unroll
      for (int j = 0; j < n; ++j) {
        if (keep(j)) {
          const uint32_t k = key_at(j);
          if (round == 0 || (k >> (shift + 8)) == prefix) add_one(hist, (int)((k >> shift) & 255u));
        }
      }
    } else {  // keys come from memory: eight reads are requested before the first one is used
      for (int j0 = 0; j0 < n; j0 += 8) {
        uint32_t kk[8];
        bool kp[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          kp[u] = j0 + u < n && keep(j0 + u);
          kk[u] = kp[u] ? key_at(j0 + u) : 0u;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (kp[u] && (round == 0 || (kk[u] >> (shift + 8)) == prefix)) add_one(hist, (int)((kk[u] >> shift) & 255u));
      }
    }
    __syncthreads();
    if (t < kWave) {  // the first wave finds the digit that holds the need-th largest key
      int cnt[4];
      int tot = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) { cnt[i] = hist[4 * t + i]; tot += cnt[i]; }
      int suf = tot;  // inclusive suffix sum over lanes: keys in bins >= 4*t
#pragma unroll
      for (int off = 1; off < kWave; off <<= 1) {
        const int o = __shfl_down(suf, off, kWave);
        if (t + off < kWave) suf += o;
      }
      int above = suf - tot;  // keys in strictly higher bins
#pragma unroll
      for (int i = 3; i >= 0; --i) {
        if (above < need && need <= above + cnt[i]) {
          *s_prefix = (prefix << 8) | (uint32_t)(4 * t + i);
          *s_need = need - above;
        }
        above += cnt[i];
      }
    }
    __syncthreads();
    prefix = *s_prefix;
    need = *s_need;
  }
  return prefix;
}

// Exclusive prefix of counts[v * kWaves + wave] (kVecs * kWaves counts in LDS, at most 256) for every v, and their total.
template <int kVecs, int kWaves>
__device__ __forceinline__ int wave_prefixes(const int* counts, int wave, int (&prefix)[kVecs]) {
  static_assert(kWaves == 1 || (kVecs * kWaves <= 4 * kWave && kWaves % 4 == 0), "four counts per lane");
  if constexpr (kWaves == 1) {
    int sum = 0;
#pragma unroll
    for (int v = 0; v < kVecs; ++v) { prefix[v] = sum; sum += counts[v]; }
    return sum;
  }
  const int lane = threadIdx.x % kWave;
  int4 q = make_int4(0, 0, 0, 0);
  if (4 * lane < kVecs * kWaves) q = *reinterpret_cast<const int4*>(&counts[4 * lane]);
  const int inc = wave_inclusive_scan(q.x + q.y + q.z + q.w);
  const int sub = wave % 4;
  const int pre = inc - (q.w + (sub < 3 ? q.z : 0) + (sub < 2 ? q.y : 0) + (sub < 1 ? q.x : 0));
#pragma unroll
  for (int v = 0; v < kVecs; ++v) prefix[v] = __builtin_amdgcn_readlane(pre, (v * kWaves + wave) / 4);
  return __builtin_amdgcn_readlane(inc, kWave - 1);
}

template <int kThreads>
struct SelectShared {
  static constexpr int kWaves = kThreads / kWave;
  static constexpr int kBuckets = kThreads >= 1024 ? 2048 : (kThreads >= 256 ? 1024 : 256);
  static constexpr int kMaxRank = kThreads < kMaxRankCandidates ? kThreads : kMaxRankCandidates;
  // every 16 buckets are followed by a gap of 4 so that the 16-byte reads of the scan spread over the LDS banks
  static __device__ __forceinline__ int slot(int bucket) { return bucket + ((bucket >> 4) << 2); }
  __attribute__((aligned(16))) int hist[kBuckets + kBuckets / 4];
  __attribute__((aligned(16))) int sure_cnt[4 * kWave], tie_cnt[4 * kWave];
  uint32_t cand_key[kMaxRank];
  int cand_page[kMaxRank];
  uint32_t wave_min[kWaves], wave_max[kWaves], wave_low[kWaves];
  int need, ncand;
  uint32_t prefix;
};

// The bucket that holds the kb-th largest counted key, how many of its keys are among the kb, and how many it has.
// Every wave scans the whole histogram for itself: lane l takes kBuckets / 64 buckets, lane 0 the topmost ones.
template <int kThreads>
__device__ __forceinline__ void boundary_bucket(const SelectShared<kThreads>& sh, int kb, int& bstar, int& need, int& ncand) {
  using Sh = SelectShared<kThreads>;
  constexpr int kPerLane = Sh::kBuckets / kWave;
  int cnt[kPerLane];
  const int b0 = (kWave - 1 - (int)(threadIdx.x % kWave)) * kPerLane;
  int tot = 0;
#pragma unroll
  for (int i = 0; i < kPerLane; i += 4) {
    const int4 q = *reinterpret_cast<const int4*>(&sh.hist[Sh::slot(b0 + i)]);
    cnt[i] = q.x; cnt[i + 1] = q.y; cnt[i + 2] = q.z; cnt[i + 3] = q.w;
    tot += q.x + q.y + q.z + q.w;
  }
  const int inc = wave_inclusive_scan(tot);
  int above = inc - tot, my_b = 0, my_need = 0, my_n = 0;
  const int src = __ffsll(__ballot(above < kb && kb <= inc)) - 1;  // exactly one lane
#pragma unroll
  for (int i = kPerLane - 1; i >= 0; --i) {
    if (above < kb) { my_b = b0 + i; my_need = kb - above; my_n = cnt[i]; }  // the last one that stays true
    above += cnt[i];
  }
  bstar = __builtin_amdgcn_readlane(my_b, src);
  need = __builtin_amdgcn_readlane(my_need, src);
  ncand = __builtin_amdgcn_readlane(my_n, src);
}

// Where the buckets lie: linear between the scores of the keys kmin and kmax (see linear_bucket).
struct BucketMap { float lo, scale; };
__device__ __forceinline__ BucketMap bucket_map(uint32_t kmin, uint32_t kmax, int n_buckets) {
  BucketMap m = {0.f, 0.f};
  if (kmin < kmax) {  // at least two distinct finite keys to tell apart
    m.lo = ordered_to_float(kmin);
    const float range = ordered_to_float(kmax) - m.lo;
    if (range > 0.f && range < 3.0e38f) m.scale = (float)(n_buckets - 1) / range;
    if (!(m.scale < 3.0e38f)) m.scale = 0.f;  // a denormal range: leave everything in one bucket
  }
  return m;
}

// The selection proper over keys in registers: thread t holds kVecs groups of kPer keys; in the order (group, thread,
// key inside the group) the pages ascend. Keys below T0 (>= 1) are not selected, at least kb keys are not below it.
// emit(at, j): the page of this thread's key j is the at-th selected one, in page order.
// The histogram in `sh` is zero and sh.ncand is 0. All threads call it.
template <int kThreads, int kVecs, int kPer, typename PageOf, typename Emit>
__device__ __forceinline__ void select_keys(const uint32_t (&key)[kVecs * kPer], PageOf page_of, uint32_t T0, BucketMap map,
                                            int kb, Emit emit, SelectShared<kThreads>& sh) {
  using Sh = SelectShared<kThreads>;
  constexpr int kWaves = Sh::kWaves, kBuckets = Sh::kBuckets, kMaxRank = Sh::kMaxRank, kItems = kVecs * kPer;
  const int t = threadIdx.x, lane = t % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(t / kWave);

  // ---- 1. histogram; the bucket of every counted key (-1: not counted) stays in registers unless the keys take most
  // (32 keys per thread, 128 rows x 24000 pages, k = 1025: 19.8 us, 23.0 with buckets made three times)
  constexpr bool kKeepBuckets = kItems <= 32;
  int bucket_reg[kKeepBuckets ? kItems : 1];
  auto make_bucket = [&](int j) { return key[j] >= T0 ? linear_bucket(key[j], map.lo, map.scale, kBuckets) : -1; };
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int bk = make_bucket(j);
    if (bk >= 0) {
      if (map.scale == 0.f) add_one(sh.hist, Sh::slot(bk));  // uniform; all finite keys share one bucket
      else atomicAdd(&sh.hist[Sh::slot(bk)], 1);
    }
    if constexpr (kKeepBuckets) bucket_reg[j] = bk;
  }
  auto bucket = [&](int j) {
    if constexpr (kKeepBuckets) return bucket_reg[j];
    else return make_bucket(j);
  };
  __syncthreads();
  // need: how many of the boundary bucket's ncand keys are selected
  int bstar, need, ncand;
  boundary_bucket<kThreads>(sh, kb, bstar, need, ncand);

  // ---- 2. candidates of the boundary bucket, and surely selected pages per (group, wave)
#pragma unroll
  for (int v = 0; v < kVecs; ++v) {
    int n = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int j = kPer * v + i, bk = bucket(j);
      n += __popcll(__ballot(bk > bstar));
      if (bk == bstar && ncand <= kMaxRank) {
        const int at = atomicAdd(&sh.ncand, 1);
        sh.cand_key[at] = key[j];
        sh.cand_page[at] = page_of(j);
      }
    }
    if (lane == 0) sh.sure_cnt[v * kWaves + wave] = n;
  }
  __syncthreads();
  int place[kVecs];  // output index of the first selected page of (group v, this wave)

  if (ncand > kMaxRank) {  // a degenerate row (many equal scores, or a range that the buckets cannot resolve)
    const uint32_t T = radix_threshold<kThreads, kItems>(
        kItems, [&](int j) { return key[j]; }, [&](int j) { return bucket(j) == bstar; }, need, sh.hist, &sh.prefix,
        &sh.need);
    // need: how many keys equal to T are taken, from the lowest page up
#pragma unroll
    for (int v = 0; v < kVecs; ++v) {
      int n = 0, e = 0;
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        n += __popcll(__ballot(key[kPer * v + i] > T));
        e += __popcll(__ballot(key[kPer * v + i] == T));
      }
      if (lane == 0) { sh.sure_cnt[v * kWaves + wave] = n; sh.tie_cnt[v * kWaves + wave] = e; }
    }
    __syncthreads();
    int ties[kVecs];
    wave_prefixes<kVecs, kWaves>(sh.sure_cnt, wave, place);
    wave_prefixes<kVecs, kWaves>(sh.tie_cnt, wave, ties);
#pragma unroll
    for (int v = 0; v < kVecs; ++v) {
      int sure_b = place[v], tie_b = ties[v];
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        sure_b = lanes_before(__ballot(key[kPer * v + i] > T), sure_b);
        tie_b = lanes_before(__ballot(key[kPer * v + i] == T), tie_b);
      }
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        const int j = kPer * v + i;
        if (key[j] > T) {
          emit(min(tie_b, need) + sure_b++, j);
        } else if (key[j] == T) {
          if (tie_b < need) emit(sure_b + tie_b, j);
          ++tie_b;
        }
      }
    }
    return;
  }

  // ---- exact rank of the candidates by (key, page): the last selected one has key T and page tpage
  uint32_t T;
  int tpage;
  wave_prefixes<kVecs, kWaves>(sh.sure_cnt, wave, place);
  int first_page[kVecs];  // page of (group v, this wave, lane 0): candidates before it lie in earlier groups or waves
#pragma unroll
  for (int v = 0; v < kVecs; ++v) first_page[v] = __builtin_amdgcn_readfirstlane(page_of(kPer * v));
  if (ncand <= kWave) {  // one candidate per lane, every wave for itself
    const uint32_t mk = lane < ncand ? sh.cand_key[lane] : 0u;
    const int mi = lane < ncand ? sh.cand_page[lane] : 0x7fffffff;
    int rank = 0;
    for (int j = 0; j < ncand; ++j) {
      const uint32_t kj = (uint32_t)__builtin_amdgcn_readlane((int)mk, j);
      const int ij = __builtin_amdgcn_readlane(mi, j);
      rank += (kj > mk) || (kj == mk && ij < mi);
    }
    const bool sel = lane < ncand && rank < need;
    const int src = __ffsll(__ballot(lane < ncand && rank == need - 1)) - 1;
    T = (uint32_t)__builtin_amdgcn_readlane((int)mk, src);
    tpage = __builtin_amdgcn_readlane(mi, src);
#pragma unroll
    for (int v = 0; v < kVecs; ++v) place[v] += __popcll(__ballot(sel && mi < first_page[v]));
  } else {
    if (t < ncand) {
      const uint32_t mk = sh.cand_key[t];
      const int mi = sh.cand_page[t];
      int rank = 0;
#pragma unroll 8
      for (int j = 0; j < ncand; ++j) rank += (sh.cand_key[j] > mk) || (sh.cand_key[j] == mk && sh.cand_page[j] < mi);
      if (rank == need - 1) { sh.prefix = mk; sh.need = mi; }
    }
    __syncthreads();
    T = sh.prefix;
    tpage = sh.need;
    for (int j0 = 0; j0 < ncand; j0 += kWave) {
      const uint32_t mk = j0 + lane < ncand ? sh.cand_key[j0 + lane] : 0u;
      const int mi = j0 + lane < ncand ? sh.cand_page[j0 + lane] : 0x7fffffff;
      const bool sel = mk > T || (mk == T && mi <= tpage);
#pragma unroll
      for (int v = 0; v < kVecs; ++v) place[v] += __popcll(__ballot(sel && mi < first_page[v]));
    }
  }

  // ---- 3. the selected pages, in page order
#pragma unroll
  for (int v = 0; v < kVecs; ++v) {
    bool sel[kPer];
    int at = place[v];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int j = kPer * v + i;
      sel[i] = key[j] > T || (key[j] == T && page_of(j) <= tpage);
      at = lanes_before(__ballot(sel[i]), at);
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      if (sel[i]) emit(at++, kPer * v + i);
  }
}

// The keys of a row of P pages in registers: kVecs loads of kPer (one or four) scores per thread, thread t holds the pages
// row_page(v * kPer + i) = (v * kThreads + t) * kPer + i, so every load of a wave is 256 B or 1 KiB of consecutive scores.
template <int kThreads, int kPer>
__device__ __forceinline__ int row_page(int j) { return ((j / kPer) * kThreads + (int)threadIdx.x) * kPer + j % kPer; }

// Keys of four scores, of which the first n are pages of the row.
__device__ __forceinline__ void keys_of(const float4& raw, int n, uint32_t* key) {
  key[0] = n > 0 ? score_key(raw.x) : 0u;
  key[1] = n > 1 ? score_key(raw.y) : 0u;
  key[2] = n > 2 ? score_key(raw.z) : 0u;
  key[3] = n > 3 ? score_key(raw.w) : 0u;
}

// The last `recent` pages (at most kb of them) take the largest key there is (above +inf), so they outrank every score.
template <int kThreads, int kVecs, int kPer>
__device__ __forceinline__ void force_recent_keys(uint32_t (&key)[kVecs * kPer], int P, int kb, int recent) {
  if (recent > 0) {
    const int forced_from = P - min(recent, kb);
#pragma unroll
    for (int j = 0; j < kVecs * kPer; ++j) {
      const int p = row_page<kThreads, kPer>(j);
      if (p >= forced_from && p < P) key[j] = kKeyForced;
    }
  }
}

// The bound T0 and the buckets for a row of P pages, kb of them to be selected (kb < P); zeroes the histogram and sh.ncand.
template <int kThreads, int kVecs, int kPer>
__device__ __forceinline__ uint32_t bound_row(const uint32_t (&key)[kVecs * kPer], int P, int kb, BucketMap& map,
                                              SelectShared<kThreads>& sh) {
  using Sh = SelectShared<kThreads>;
  constexpr int kWaves = Sh::kWaves, kItems = kVecs * kPer, kBuckets = Sh::kBuckets;
  const int t = threadIdx.x, lane = t % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
  // The row's smallest and largest finite key, and a lower bound T0 of the k-th key: the smallest of the maxima of
  // disjoint groups of keys, of which there are at least kb. Groups are the keys of 2^n threads, as many as leave
  // enough groups; threads without a page do not count.
  uint32_t kmin = 0xffffffffu, kmax = 0u, low = 0u;
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const bool finite = key[j] > kKeyNegInf && key[j] < kKeyPosInf;
    kmin = min(kmin, finite ? key[j] : 0xffffffffu);
    kmax = max(kmax, finite ? key[j] : 0u);
    low = max(low, key[j]);
  }
  {
    const int busy = min(kThreads, (P + kPer - 1) / kPer);  // threads with a page
    auto merge = [&](int lanes, uint32_t other) { if (lanes * kb <= busy) low = max(low, other); };
    merge(2, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)low, kDppXor1, 0xf, 0xf, true));
    merge(4, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)low, kDppXor2, 0xf, 0xf, true));
    merge(8, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)low, kDppHalfMirror, 0xf, 0xf, true));
    merge(16, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)low, kDppMirror, 0xf, 0xf, true));
    if (kb > busy) low = 0u;
    else if (t >= busy) low = 0xffffffffu;
  }
  kmin = wave_allreduce_minmax<false>(kmin);
  kmax = wave_allreduce_minmax<true>(kmax);
  low = wave_allreduce_minmax<false>(low);
  if (lane == 0) { sh.wave_min[wave] = kmin; sh.wave_max[wave] = kmax; sh.wave_low[wave] = low; }
  for (int i = t; i < kBuckets + kBuckets / 4; i += kThreads) sh.hist[i] = 0;
  if (t == 0) sh.ncand = 0;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    kmin = min(kmin, sh.wave_min[w]); kmax = max(kmax, sh.wave_max[w]); low = min(low, sh.wave_low[w]);
  }
  const uint32_t T0 = max(low, 1u);
  if (T0 > kKeyNegInf && T0 < kKeyPosInf) kmin = T0;
  map = bucket_map(kmin, kmax, kBuckets);
  return T0;
}

// Selection by re-reading the row in every pass (it stays in L2): histogram between the row's smallest and largest
// finite key, candidates, compaction. Thread t owns the pages t, t + threads, t + 2*threads, ... so that every read of the
// row is coalesced, eight reads at a time. The compaction walks the row in blocks of `threads` consecutive pages and
// places each selected page by a ballot prefix inside its wave, the wave totals of the block (LDS) and the running
// totals of the blocks before it, which keeps the output in ascending page order and takes keys tied with the k-th from
// the lowest page upward. emit(at, page): the page is the at-th selected one.
// The histogram in `sh` is zero and sh.ncand is 0. All threads call it.
template <int kThreads, typename KeyOf, typename Emit>
__device__ __forceinline__ void select_reread(KeyOf key_of, int P, int kb, BucketMap map, Emit emit,
                                              SelectShared<kThreads>& sh) {
  using Sh = SelectShared<kThreads>;
  constexpr int kWaves = Sh::kWaves, kBuckets = Sh::kBuckets, kMaxRank = Sh::kMaxRank;
  const int t = threadIdx.x, lane = t % kWave, wave = t / kWave;
  const int ipt = (P + kThreads - 1) / kThreads;  // strided items per thread; the last ones may fall past P
  auto for_each_key = [&](auto f) {               // f(page, key) for every page this thread owns
    for (int j0 = 0; j0 < ipt; j0 += 8) {
      uint32_t kk[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int page = (j0 + u) * kThreads + t;
        kk[u] = page < P ? key_of(page) : 0u;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int page = (j0 + u) * kThreads + t;
        if (page < P) f(page, kk[u]);
      }
    }
  };

  // ---- 1. histogram
  auto bucket_of = [&](uint32_t k) { return linear_bucket(k, map.lo, map.scale, kBuckets); };
  if (map.scale == 0.f) for_each_key([&](int, uint32_t k) { add_one(sh.hist, Sh::slot(bucket_of(k))); });
  else for_each_key([&](int, uint32_t k) { atomicAdd(&sh.hist[Sh::slot(bucket_of(k))], 1); });
  __syncthreads();
  int bstar, need, ncand;  // need: how many of the boundary bucket's ncand keys are selected
  boundary_bucket<kThreads>(sh, kb, bstar, need, ncand);

  // ---- 2. exact threshold inside the boundary bucket: key T and how many keys equal to T to take
  uint32_t T;
  if (ncand <= kMaxRank) {
    for_each_key([&](int page, uint32_t k) {
      if (bucket_of(k) == bstar) {
        const int at = atomicAdd(&sh.ncand, 1);
        sh.cand_key[at] = k;
        sh.cand_page[at] = page;
      }
    });
    __syncthreads();
    if (t < ncand) {
      const uint32_t mk = sh.cand_key[t];
      const int mi = sh.cand_page[t];
      int rank = 0, greater = 0;
      for (int j = 0; j < ncand; ++j) {
        const uint32_t k = sh.cand_key[j];
        greater += k > mk;
        rank += (k > mk) || (k == mk && sh.cand_page[j] < mi);
      }
      if (rank == need - 1) { sh.prefix = mk; sh.need = need - greater; }
    }
    __syncthreads();
    T = sh.prefix;
    need = sh.need;
  } else {
    T = radix_threshold<kThreads, 0>(
        ipt, [&](int j) { return key_of(j * kThreads + t); },
        [&](int j) { return j * kThreads + t < P && bucket_of(key_of(j * kThreads + t)) == bstar; }, need, sh.hist,
        &sh.prefix, &sh.need);
  }

  // ---- 3. compaction in page order. "gt": above the k-th key; "eq": equal to it.
  int gt_run = 0, eq_run = 0;  // such pages in the blocks already walked
  constexpr int kAhead = 8;    // blocks whose keys are read together, ahead of the barriers that walk them
  for (int base0 = 0, it = 0; base0 < P; base0 += kAhead * kThreads) {
    uint32_t kk[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int page = base0 + u * kThreads + t;
      kk[u] = page < P ? key_of(page) : 0u;
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u, ++it) {
      const int page = base0 + u * kThreads + t;
      if (base0 + u * kThreads >= P) break;  // uniform
      const bool gt = page < P && kk[u] > T, eq = page < P && kk[u] == T;
      const unsigned long long bg = __ballot(gt), be = __ballot(eq);
      int* wave_gt = sh.sure_cnt + (it & 1) * kWaves;
      int* wave_eq = sh.tie_cnt + (it & 1) * kWaves;
      if (lane == 0) { wave_gt[wave] = __popcll(bg); wave_eq[wave] = __popcll(be); }
      __syncthreads();  // the buffers alternate, so one barrier per block is enough
      int gt_before = lanes_before(bg, gt_run), eq_before = lanes_before(be, eq_run);
      int gt_block = 0, eq_block = 0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const int g = wave_gt[w], e = wave_eq[w];
        gt_before += w < wave ? g : 0;
        eq_before += w < wave ? e : 0;
        gt_block += g;
        eq_block += e;
      }
      if (gt) emit(gt_before + min(eq_before, need), page);
      else if (eq && eq_before < need) emit(gt_before + eq_before, page);
      gt_run += gt_block;
      eq_run += eq_block;
    }
  }
}

}  // namespace
}  // namespace unique
