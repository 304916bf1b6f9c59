// Attention over one chunk of a row's page list, by one workgroup of four waves: the device code that the decode kernels
// (decode.hip) and the kernels that also make the list (step.hip) share. The caller says which physical page an entry of
// the chunk is and how many tokens of it count.
#pragma once
#include "device_utils.hpp"
#include "kernels.hpp"
#include "split_plan.hpp"

namespace unique {
namespace {

constexpr float kNegBig = -1.0e30f;  // finite stand-in for "no logit seen yet"
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// With a single chunk per row there is nothing to merge: the partial kernel writes the attention output
// itself, with the arithmetic of the merge kernel (a scale of exp2(0) = 1), so the result is the same bits.
template <typename T>
__device__ __forceinline__ void write_final(const CacheView& c, T* out, float* lse_out, int b, int h, int d, int D,
                                            float o, float M, float L) {
  const bool any = L > 0.f;
  store_elem(out + ((int64_t)b * c.H + h) * D + d, any ? o / L : 0.f);
  if (lse_out && d == 0) lse_out[(int64_t)b * c.H + h] = any ? (M + log2f(L)) * kLn2 : -INFINITY;
}

// The chunk of a workgroup. With SplitPlan::rotate the split is the slowest grid index, so that empty chunks come last, and
// from one split to the next the rows move on by a head and a sequence: the chunks of a row, which may be the only long
// one, then lie on different XCDs (workgroups are dealt to the 8 of them in turn) and different compute units there.
// Selects instead of a branch: with a branch the kernel's arguments arrive in two round trips (0.1 us).
__device__ __forceinline__ void locate_chunk(const CacheView& c, const SplitPlan& plan, int& split, int& hkv, int& b) {
  const bool rot = plan.rotate != 0;
  split = rot ? blockIdx.z : blockIdx.x;
  const int by = rot ? split : 0;
  hkv = ((rot ? blockIdx.x : blockIdx.y) + by) & (c.Hkv - 1);  // a power of two
  b = (rot ? blockIdx.y : blockIdx.z) + (by & (plan.rotate - 1));
  b -= b >= c.B ? c.B : 0;
}

// Where a workgroup's results go: the chunk's part of the workspace, or the output if the row has one chunk.
template <typename T>
struct ChunkOut {
  float* part_o;   // [slots][G][D], a slot per chunk
  float* part_ml;  // [slots][G][2]
  T* out;          // written directly when num_splits == 1
  float* lse_out;
  int num_splits;
};

// A chunk: entries [begin, end) of the list of sequence b and KV head hkv, the sequence's length, and the slot of its results.
struct Chunk {
  int hkv, b, begin, end, N;
  int64_t slot;
};

// An empty list: the output is defined as zero, the lse as -inf.
template <typename T, int D, int G>
__device__ __forceinline__ void write_empty(const CacheView& c, const ChunkOut<T>& to, int b, int hkv) {
  if (to.num_splits == 1) {
    for (int idx = threadIdx.x; idx < G * D; idx += kDecWaves * kWave)
      write_final(c, to.out, to.lse_out, b, hkv * G + idx / D, idx % D, D, 0.f, 0.f, 0.f);
  }
}

template <typename T, int D, int G>
struct DecodeShared {  // the waves' results, merged at the end; bf16 caches: output rows are parts times heads
  static constexpr int kSlots = sizeof(T) == 4 ? G : (G == 8 ? 16 : 3 * G);
  __attribute__((aligned(16))) float acc[kDecWaves][kSlots][D];
  float m[kDecWaves][G], l[kDecWaves][G];
};

// The waves' results, all in `sh`, become the chunk's: partial results, or the output of a row with one chunk. A thread takes as many
// consecutive channels of a head as there are: a loop over single ones repeated the scales and waited for the LDS twice with four heads of
// 128 channels (a step of 32K tokens 18.5 / 18.3 us, 12 x 50K with eight heads 61.3 / 60.8, the toy model 10.8 / 10.6). It is written as a loop of one
// turn all the same: with an early return in its place every instance becomes longer, and one-kernel steps of two heads took 9.7 us for 9.6 (10 x 40 pages) and
// 9.9 for 9.8 (25 x 81), the step of 32K tokens 16.1 for 15.9 to 16.1.
template <typename T, int D, int G>
__device__ __forceinline__ void finish_chunk(const CacheView& c, const Chunk& k, const ChunkOut<T>& to, const DecodeShared<T, D, G>& sh) {
  constexpr int kSlots = DecodeShared<T, D, G>::kSlots;
  constexpr int kPer = G * D <= kDecWaves * kWave ? 1 : G * D / (kDecWaves * kWave);
  static_assert(kPer <= 4, "a 16-byte access");
  typedef float vec_t __attribute__((ext_vector_type(kPer)));
  for (int at = threadIdx.x * kPer; at < G * D; at += kDecWaves * kWave * kPer) {  // once
    const int g = at / D, d = at % D;
    float M = sh.m[0][g];
#pragma unroll
    for (int w = 1; w < kDecWaves; ++w) M = fmaxf(M, sh.m[w][g]);
    float o[kPer], L = 0.f;
#pragma unroll
    for (int i = 0; i < kPer; ++i) o[i] = 0.f;
#pragma unroll
    for (int w = 0; w < kDecWaves; ++w) {
      const float sc = fast_exp2(sh.m[w][g] - M);
      vec_t ow = *reinterpret_cast<const vec_t*>(&sh.acc[w][g][d]);
#pragma unroll
      for (int r = G + g; r < kSlots; r += G) ow += *reinterpret_cast<const vec_t*>(&sh.acc[w][r][d]);
#pragma unroll
      for (int i = 0; i < kPer; ++i) o[i] = fmaf(ow[i], sc, o[i]);
      L = fmaf(sh.l[w][g], sc, L);
    }
    if (to.num_splits == 1) {
#pragma unroll
      for (int i = 0; i < kPer; ++i) write_final(c, to.out, to.lse_out, k.b, k.hkv * G + g, d + i, D, o[i], M, L);
    } else {
      vec_t out;
#pragma unroll
      for (int i = 0; i < kPer; ++i) out[i] = o[i];
      *reinterpret_cast<vec_t*>(&to.part_o[(k.slot * G + g) * D + d]) = out;
      if (d == 0) {
        to.part_ml[(k.slot * G + g) * 2 + 0] = M;
        to.part_ml[(k.slot * G + g) * 2 + 1] = L;
      }
    }
  }
}

// ---- fp32 caches: vector ALUs ----
// kNT: K and V are read with non-temporal loads (a launch that streams more than the caches hold). It is a template
// parameter because the compiler merges the two loads of a run-time choice into a plain one.
// us before (predicated loads, run-time choice) and now: 128 rows x 128 pages of 16 KB, G = 4 62.9 / 45.8 (5.9 TB/s);
// all of 4 x 32768 tokens, G = 8 224 / 197; 2 rows x 16 pages of 8 KB 7.8 / 6.4.
template <int D, int S, int G, bool kNT, typename Lookup>
__device__ __forceinline__ void decode_chunk(const CacheView& c, const float* __restrict__ q, const Chunk& k, int wave, int lane, Lookup lookup,
                                             float scale_log2, const ChunkOut<float>& to, DecodeShared<float, D, G>& sh) {
  using T = float;
  constexpr int kVec = Elem<T>::kVec;
  constexpr int kLanesPerTok = D / kVec;
  constexpr int kTokPerLoad = kWave / kLanesPerTok;
  constexpr int kLoads = S / kTokPerLoad;                       // wave-wide loads per page (K or V)
  constexpr int kTileLoads = kLoads < 4 ? kLoads : 4;           // loads handled per pipeline stage
  constexpr int kTilesPerPage = kLoads / kTileLoads;
  constexpr int kBuffers = 2;  // register tiles per wave (three and four measured no faster)
  static_assert(S % kTokPerLoad == 0 && kLoads % kTileLoads == 0, "page size / element type combination");
  // Eight heads are bound by the vector ALUs, and four nearly, so their sums over lanes 16 and 32 apart go through the LDS. us with row swaps /
  // so, D = 128, pages of 16: 8 heads, dense 1 x 11828 pages 284 / 270 (275 with the sums of the logits alone), steps of 53 x 891, 4 KV heads, k = 159
  // 148.4 / 145.2, 36 x 96, 17 39.7 / 37.7; 4 heads 36 x 96, 17 29.1 / 28.5, 25 x 862, 336 215.3 / 212.6; 1 and 2 the same. Eight heads over short chunks of cut
  // rows lose (20 x 9000 pages of 8, k = 64 19.4 / 20.0), which the same instances cannot tell. A token of 64 channels is in 16 lanes,
  // so that only the end has such sums, a chain of them: the toy model 10.1 / 10.4, 1 x 2048 pages, 8 heads 16.5 / 16.8, 40 x 300 the same.
  constexpr bool kLds = G >= 4 && D == 128;

  const int hkv = k.hkv, b = k.b, begin = k.begin, end = k.end;

  const int tr = lane / kLanesPerTok, ch = lane % kLanesPerTok;

  const T* q_row = q + ((int64_t)b * c.H + hkv * G) * D + ch * kVec;  // this lane's chunk of the group's first query
  float qv[G][kVec];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    load_vec(q_row + g * D, qv[g]);
#pragma unroll
    for (int i = 0; i < kVec; ++i) qv[g][i] *= scale_log2;
  }

  float m[G], l[G], acc[G][kVec];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    m[g] = kNegBig;
    l[g] = 0.f;
#pragma unroll
    for (int i = 0; i < kVec; ++i) acc[g][i] = 0.f;
  }

  const T* kc = reinterpret_cast<const T*>(c.k_cache);
  const T* vc = reinterpret_cast<const T*>(c.v_cache);
  const int64_t lane_off = ch * kVec;

  // entries of this chunk are dealt to the waves round-robin; a wave looks up 64 of them at a time
  for (int e0 = begin + wave; e0 < end; e0 += kDecWaves * kWave) {
    int my_phys = 0, my_ntok = 0;
    if (e0 + lane * kDecWaves < end) lookup(e0 + lane * kDecWaves, e0 == begin + wave, my_phys, my_ntok);
    const int n_ent = min(kWave, (end - e0 + kDecWaves - 1) / kDecWaves);
    const int n_tiles = n_ent * kTilesPerPage;

    // A ring of register tiles, one being consumed and the others in flight. Loads are unconditional -- a slot without a
    // token reads the first query instead, whose probability is zero -- so that every wait is exact (see the
    // matrix-core kernel; with predicated loads the compiler waits for all of them before each tile).
    Raw16 kb[kBuffers][kTileLoads], vb[kBuffers][kTileLoads];
    int left[kBuffers];  // tokens of the page from this lane group's first slot on
    auto issue = [&](int it, Raw16(&kd)[kTileLoads], Raw16(&vd)[kTileLoads], int& rest) {
      const int ent = min(it / kTilesPerPage, kWave - 1);
      const int phys = __builtin_amdgcn_readlane(my_phys, ent);
      const int ntok = it < n_tiles ? __builtin_amdgcn_readlane(my_ntok, ent) : 0;
      const int tok0 = (it % kTilesPerPage) * kTileLoads * kTokPerLoad + tr;
      const int64_t off = (int64_t)phys * c.kv_page_stride + (int64_t)hkv * c.kv_head_stride + (int64_t)tok0 * D + lane_off;
      rest = ntok - tok0;
#pragma unroll
      for (int j = 0; j < kTileLoads; ++j) {
        const bool valid = j * kTokPerLoad < rest;
        kd[j] = load_raw_stream(valid ? kc + off + j * kTokPerLoad * D : q_row, kNT);
        vd[j] = load_raw_stream(valid ? vc + off + j * kTokPerLoad * D : q_row, kNT);
      }
    };
    auto consume = [&](const Raw16(&kr)[kTileLoads], Raw16(&vr)[kTileLoads], int rest) {
      // logits of this lane group's tokens for the G heads
      float s[kTileLoads][G];
#pragma unroll
      for (int j = 0; j < kTileLoads; ++j) {
        float kf[kVec];
        unpack_raw(kr[j], kf, (const T*)nullptr);
#pragma unroll
        for (int g = 0; g < G; ++g) {
          float d = qv[g][0] * kf[0];
#pragma unroll
          for (int i = 1; i < kVec; ++i) d = fmaf(qv[g][i], kf[i], d);
          d = group_allreduce<kLanesPerTok, kLds>(d, OpSum());
          s[j][g] = j * kTokPerLoad < rest ? d : -INFINITY;
        }
      }
      // online softmax update, one state per lane group
      float p[kTileLoads][G];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        float mx = s[0][g];
#pragma unroll
        for (int j = 1; j < kTileLoads; ++j) mx = fmaxf(mx, s[j][g]);
        const float mnew = fmaxf(m[g], mx);
        const float alpha = fast_exp2(m[g] - mnew);
        m[g] = mnew;
        float psum = 0.f;
#pragma unroll
        for (int j = 0; j < kTileLoads; ++j) {
          p[j][g] = fast_exp2(s[j][g] - mnew);
          psum += p[j][g];
        }
        l[g] = fmaf(l[g], alpha, psum);
#pragma unroll
        for (int i = 0; i < kVec; ++i) acc[g][i] *= alpha;
      }
      // A filler's value counts as zero: a query that is infinite or NaN must not reach the outputs of the other heads.
      if (__any(rest <= (kTileLoads - 1) * kTokPerLoad)) {
#pragma unroll
        for (int j = 0; j < kTileLoads; ++j)
          if (j * kTokPerLoad >= rest) vr[j] = zero_raw();
      }
#pragma unroll
      for (int j = 0; j < kTileLoads; ++j) {
        float vf[kVec];
        unpack_raw(vr[j], vf, (const T*)nullptr);
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int i = 0; i < kVec; ++i) acc[g][i] = fmaf(p[j][g], vf[i], acc[g][i]);
      }
    };

    // A page or less per wave has nothing to prefetch, and the fillers of a pipeline cost it 0.4 us (2 rounds of 8 loads: 8 rows
    // x 64 pages, D = 64 8.2 / 7.7). With 8 heads the loop suffers from the second copy of the arithmetic (4 x 32768 tokens 97 / 121).
    if (G < 8 && n_tiles == 1) {
      issue(0, kb[0], vb[0], left[0]);
      consume(kb[0], vb[0], left[0]);
      continue;
    }
#pragma unroll
    for (int u = 0; u < kBuffers - 1; ++u) issue(u, kb[u], vb[u], left[u]);
    for (int t0 = 0; t0 < n_tiles; t0 += kBuffers) {
#pragma unroll
      for (int u = 0; u < kBuffers; ++u) {
        constexpr int kAhead = kBuffers - 1;
        issue(t0 + u + kAhead, kb[(u + kAhead) % kBuffers], vb[(u + kAhead) % kBuffers], left[(u + kAhead) % kBuffers]);
        if (u == 0 || t0 + u < n_tiles) consume(kb[u], vb[u], left[u]);  // uniform
      }
    }
  }

  // merge the lane groups of the wave (they hold disjoint token subsets)
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const float M = cross_group_allreduce<kLanesPerTok, kLds>(m[g], OpMax());
    const float sc = fast_exp2(m[g] - M);
    m[g] = M;
    l[g] = cross_group_allreduce<kLanesPerTok, kLds>(l[g] * sc, OpSum());
#pragma unroll
    for (int i = 0; i < kVec; ++i) acc[g][i] = cross_group_allreduce<kLanesPerTok, kLds>(acc[g][i] * sc, OpSum());
  }

  if (tr == 0) {
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int i = 0; i < kVec; ++i) sh.acc[wave][g][ch * kVec + i] = acc[g][i];
  }
  if (lane == 0) {
#pragma unroll
    for (int g = 0; g < G; ++g) { sh.m[wave][g] = m[g]; sh.l[wave][g] = l[g]; }
  }
  __syncthreads();
  finish_chunk<float, D, G>(c, k, to, sh);
}

// ---- bf16 caches: both products of a tile of 16 tokens run on the matrix cores ----
// v_mfma_f32_16x16x32_bf16 computes D[m][n] += sum_k A[m][k] B[k][n]: lane L supplies row m = L % 16 of A and column
// n = L % 16 of B, 8 consecutive k of its 16-lane group L / 16 each, and holds D[4 * (L / 16) + i][L % 16] in register i;
// v_mfma_f32_16x16x16_bf16 is the same with 4 consecutive k.
// q.k: A = the keys of 16 token slots, B = the G query heads, repeated over the 16 columns. A lane reads, for step s, the
// 16-byte chunk 4 * s + L / 16 of its token's key, so the contraction order inside a step is whatever the hardware pairs
// up -- the same for A and B. Lane L ends up with the logits of tokens 4 * (L / 16) + i for head L % 16 % G.
// p.V: those are the four k that lane L has to supply for row L % 16 of A, so the probabilities never leave their lane.
// The probabilities stay fp32: p = hi + mid + lo, three bf16 numbers of 8 bits each, exactly; the columns of the q.k
// product are G heads times the parts, so that lane L supplies part L % 16 / G of its head (with G = 8 only two parts fit,
// the third is a second product into the rows of the first). The rows of the parts are summed at the end. An infinite value
// gives NaN, not an infinity: the lower parts of p are often zero (inputs are assumed finite).
// V is read so that lane L holds tokens 4 * (L / 16) + j, channels kVB * (L % 16) + e: the halves of the four tokens'
// words are the B operand of channel e without any exchange between lanes.
// On the vector ALUs the p.V product alone was 32 * G + 32 instructions per tile at D = 128, which made G = 8 issue-bound.
// Kernel us before and now, with the chunks as they were: G = 8, 96 rows x 200 pages of 8 KB 43.3 / 36.0; G = 4,
// 128 x 256 47.0 / 45.8, 256 x 64 pages of 16 KB 47.3 / 44.4 (6.05 TB/s), 640 x 64 pages of 4 KB 36.7 / 34.6. G = 1 and 2,
// which use 3 and 6 of the 16 output rows, gain little but lose nothing, although G = 1 at D = 128 now has two waves per
// SIMD and had three: 640 x 64 pages of 8 KB, G = 1 61.6 / 60.7, G = 2 62.4 / 60.8 (8 rows x 64 pages, G = 1: 8.5 / 8.8).
// Profiling build (-DUNIQUE_DEC_STAMPS, a second library next to the product one): every wave of the matrix-core
// kernel records the 100 MHz wall clock at kernel entry, once its page ids are resolved, after its first tile, at
// the end of its loop and after its stores, after every tile, and the compute unit it ran on, into a device array
// that unique_debug_dec_stamps() hands out; unique_debug_gather_probe() (decode.hip) is the bare memory access of the
// kernel. The product build has none of it.
#ifdef UNIQUE_DEC_STAMPS
constexpr int kStampSlots = 32, kStampWaves = 1 << 14;
__device__ unsigned long long g_dec_stamps[kStampWaves][kStampSlots];
#define DEC_STAMP(slot)                                                                                         \
  do {                                                                                                          \
    const int64_t sw_ = chunk_slot * kDecWaves + wave;                                                              \
    if (lane == 0 && sw_ < kStampWaves) g_dec_stamps[sw_][slot] = wall_clock64();                               \
  } while (0)
// the stamp is taken only once `value` (a 32-bit register) has been produced
#define DEC_STAMP_AFTER(slot, value)                 \
  do {                                               \
    asm volatile("" ::"v"(value) : "memory");        \
    DEC_STAMP(slot);                                 \
  } while (0)
#else
#define DEC_STAMP(slot) do {} while (0)
#define DEC_STAMP_AFTER(slot, value) do {} while (0)
#endif

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ bf16x8_t as_bf16x8(const Raw16& r) {
  return __builtin_bit_cast(bf16x8_t, r.v);
}
// the low / the high halves of two words, `a` in the lower half of the result
__device__ __forceinline__ uint32_t pack_lo(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ uint32_t pack_hi(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }
__device__ __forceinline__ s16x4_t as_s16x4(uint32_t a, uint32_t b) {
  const u32x2_t v = {a, b};
  return __builtin_bit_cast(s16x4_t, v);
}
// x without the lower 16 bits of its mantissa, i.e. the bf16 number in its upper half
__device__ __forceinline__ float bf16_part(float x) { return __uint_as_float(__float_as_uint(x) & 0xffff0000u); }

// Reduction over the four 16-lane groups of a wave (lanes with the same L % 16); every lane gets the result.
template <typename Op>
__device__ __forceinline__ float rows_allreduce(float x, Op op) {
  return with_lane_xor32(with_lane_xor16(x, op), op);
}

// One value row chunk of kVB bf16 elements (16 or 8 bytes) as raw words.
template <int kVB, bool kNT>
__device__ __forceinline__ void load_v(const bf16_t* p, uint32_t (&out)[kVB / 2]) {
  if constexpr (kVB == 8) {
    const Raw16 r = load_raw_stream(p, kNT);
    out[0] = r.v.x; out[1] = r.v.y; out[2] = r.v.z; out[3] = r.v.w;
  } else {
    const u32x2_t* src = reinterpret_cast<const u32x2_t*>(p);
    u32x2_t r;
    if constexpr (kNT) r = __builtin_nontemporal_load(src);
    else r = *src;
    out[0] = r.x; out[1] = r.y;
  }
}

// Register tiles per wave: one being consumed, the others in flight. Three are no faster (128 x 256 pages 46.4 us
// against 45.8, 256 x 64 pages of 16 KB 44.9 against 44.4).
constexpr int kDecBuffers = 2;

// kNT: K and V are read with non-temporal loads (a launch that streams more than the caches hold).
template <int D, int S, int G, bool kNT, typename Lookup>
__device__ __forceinline__ void decode_chunk(const CacheView& c, const bf16_t* __restrict__ q, const Chunk& k, int wave, int lane, Lookup lookup,
                                             float scale_log2, const ChunkOut<bf16_t>& to, DecodeShared<bf16_t, D, G>& sh) {
  constexpr int kVec = 8;
  constexpr int kTile = 16;                          // token slots per MFMA tile
  constexpr int kSteps = D / 32;                     // q.k steps (and K loads per lane) per tile
  constexpr int kVB = D / 16;                        // channels of a value row per lane
  constexpr int kSlots = G == 8 ? 16 : 3 * G;        // output rows in use: parts times heads
  constexpr float kRoom = 6.f;                       // log2: how far above the largest logit the reference is put
  static_assert(G <= 8, "at most 8 query heads per KV head");

  const int hkv = k.hkv, b = k.b, begin = k.begin, end = k.end;
#ifdef UNIQUE_DEC_STAMPS
  const int64_t chunk_slot = k.slot;
#endif

  const int kt = lane % 16, kg = lane / 16;  // column (token slot of K, head and part of p, channel block of V); lane group
  const int part = kt / G;                   // which part of its head's probabilities this lane supplies

  // B operand of q.k: query head kt % G, the 8 elements of chunk 4*s + kg
  const bf16_t* q_row = q + ((int64_t)b * c.H + hkv * G) * D;  // first query row of the group
  bf16x8_t qa[kSteps];
#pragma unroll
  for (int s = 0; s < kSteps; ++s) qa[s] = as_bf16x8(load_raw(q_row + (int64_t)(kt % G) * D + (4 * s + kg) * kVec));

  // Softmax state of head kt % G. The reference m, the same in all lanes of a head, is put kRoom above the largest logit and
  // only moves when a logit exceeds it: most tiles need neither the maximum over the lanes nor a rescaled output, and
  // probabilities relative to it are at most 1, so that their products with V stay in its range. l is this lane's
  // part of the sum.
  float m = kNegBig, l = 0.f;
  f32x4_t acc[kVB];  // acc[e][i]: output row 4 * kg + i (head row % G), channel kVB * kt + e
#pragma unroll
  for (int e = 0; e < kVB; ++e) acc[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const bf16_t* kc = reinterpret_cast<const bf16_t*>(c.k_cache);
  const bf16_t* vc = reinterpret_cast<const bf16_t*>(c.v_cache);
  const int64_t head_off = (int64_t)hkv * c.kv_head_stride;
  const int64_t page_stride = c.kv_page_stride;

  for (int e0 = begin + wave; e0 < end; e0 += kDecWaves * kWave) {
    int my_phys = 0, my_ntok = 0;
    if (e0 + lane * kDecWaves < end) lookup(e0 + lane * kDecWaves, e0 == begin + wave, my_phys, my_ntok);
    const int n_ent = min(kWave, (end - e0 + kDecWaves - 1) / kDecWaves);
    const int n_tiles = (n_ent * S + kTile - 1) / kTile;
    DEC_STAMP_AFTER(1, my_phys);  // page ids resolved (list entry and page-table entry arrived)

    // slot gs (counted over the wave's entries) -> entry gs / S, token gs % S. Entries at or beyond n_ent
    // were never looked up and carry ntok = 0; so does every slot of a tile at or beyond n_tiles.
    auto slot_info = [&](int tile, int slot, int& phys, int& ntok, int& tok) {
      const int gs = tile * kTile + slot;
      tok = gs % S;
      if constexpr (S >= kTile) {  // one entry per tile: uniform, scalar broadcast
        const int ent = min(tile / (S / kTile), kWave - 1);
        phys = __builtin_amdgcn_readlane(my_phys, ent);
        ntok = tile < n_tiles ? __builtin_amdgcn_readlane(my_ntok, ent) : 0;
      } else {                     // two pages share a tile: per-lane lookup
        const int ent = min(gs / S, kWave - 1);
        phys = __shfl(my_phys, ent, kWave);
        ntok = tile < n_tiles ? __shfl(my_ntok, ent, kWave) : 0;
      }
    };

    // kDecBuffers register tiles: while one is consumed, the loads of the following kDecBuffers - 1 are in flight,
    // so a wave is not paced by one memory round trip per tile. Every load is issued unconditionally -- a slot
    // that has no token (beyond a partial page, an invalid list entry, a tile past the wave's last) reads the
    // group's first query row instead, which is always cached, finite and never attended (its probability is
    // zero) -- so the pipeline is straight-line code and every wait names exactly the requests that may stay in
    // flight; with predicated loads the compiler waited for ALL outstanding loads before each tile, prefetched
    // ones included. Slots beyond a sequence's length are still never read.
    Raw16 kb[kDecBuffers][kSteps];
    uint32_t vb[kDecBuffers][4][kVB / 2];
    int kv[kDecBuffers];  // how many of the token slots 4 * kg .. 4 * kg + 3 hold a token (any value <= 0: none)
    auto issue = [&](int tile, Raw16(&kd)[kSteps], uint32_t(&vd)[4][kVB / 2], int& valid) {
      int phys, ntok, tok;
      slot_info(tile, kt, phys, ntok, tok);
      const bf16_t* kp = tok < ntok ? kc + phys * page_stride + head_off + (int64_t)tok * D + kg * kVec : q_row;
#pragma unroll
      for (int s = 0; s < kSteps; ++s) kd[s] = load_raw_stream(kp + s * (4 * kVec), kNT);
      // four consecutive token slots lie in one page
      slot_info(tile, 4 * kg, phys, ntok, tok);
      const bf16_t* vp = vc + phys * page_stride + head_off + (int64_t)tok * D + kt * kVB;
      valid = ntok - tok;
#pragma unroll
      for (int j = 0; j < 4; ++j) load_v<kVB, kNT>(j < valid ? vp + j * D : q_row, vd[j]);
    };
    auto consume = [&](const Raw16(&kr)[kSteps], const uint32_t(&vr)[4][kVB / 2], int valid) {
      f32x4_t sacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < kSteps; ++s)
        sacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(kr[s]), qa[s], sacc, 0, 0, 0);

      float x[4];  // logits of token slots 4 * kg + j relative to m, then the probabilities
#pragma unroll
      for (int j = 0; j < 4; ++j) x[j] = j < valid ? fmaf(sacc[j], scale_log2, -m) : -INFINITY;
      const float top = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
      if (__any(top > 0.f)) {
        // (from the logits themselves: m may still be kNegBig)
        float t = -INFINITY;
#pragma unroll
        for (int j = 0; j < 4; ++j) t = j < valid ? fmaxf(t, sacc[j] * scale_log2) : t;
        const float mnew = fmaxf(m, rows_allreduce(t, OpMax()) + kRoom);
        const float alpha = fast_exp2(m - mnew);
        m = mnew;
        l *= alpha;
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = j < valid ? fmaf(sacc[j], scale_log2, -m) : -INFINITY;
        // output row 4 * kg + i belongs to head (4 * kg + i) % G, whose alpha lane (4 * kg + i) % G holds
        float row_alpha[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          auto lane_alpha = [&](int n) {
            return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(alpha), n));
          };
          row_alpha[i] = lane_alpha(i % G);
          if constexpr (G == 8) row_alpha[i] = kg % 2 ? lane_alpha(4 + i) : row_alpha[i];
        }
#pragma unroll
        for (int e = 0; e < kVB; ++e)
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[e][i] *= row_alpha[i];
      }
      uint32_t pa[4], pb[4];  // this lane's part of the probabilities; pb: the third part with G = 8
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float p = fast_exp2(x[j]);
        l += p;
        const float r1 = p - bf16_part(p), r2 = r1 - bf16_part(r1);
        if constexpr (G == 8) {
          pa[j] = __float_as_uint(part == 0 ? p : r1);
          pb[j] = part == 0 ? __float_as_uint(r2) : 0u;
        } else {
          pa[j] = __float_as_uint(part == 0 ? p : (part == 1 ? r1 : r2));
        }
      }
      const s16x4_t a0 = as_s16x4(pack_hi(pa[0], pa[1]), pack_hi(pa[2], pa[3]));
      s16x4_t a1 = a0;
      if constexpr (G == 8) a1 = as_s16x4(pack_hi(pb[0], pb[1]), pack_hi(pb[2], pb[3]));
#pragma unroll
      for (int e = 0; e < kVB; ++e) {
        const int w = e / 2;
        const s16x4_t v = e % 2 == 0 ? as_s16x4(pack_lo(vr[0][w], vr[1][w]), pack_lo(vr[2][w], vr[3][w]))
                                     : as_s16x4(pack_hi(vr[0][w], vr[1][w]), pack_hi(vr[2][w], vr[3][w]));
        acc[e] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a0, v, acc[e], 0, 0, 0);
        if constexpr (G == 8) acc[e] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a1, v, acc[e], 0, 0, 0);
      }
    };

#pragma unroll
    for (int u = 0; u < kDecBuffers - 1; ++u) issue(u, kb[u], vb[u], kv[u]);
    for (int t0 = 0; t0 < n_tiles; t0 += kDecBuffers) {
#pragma unroll
      for (int u = 0; u < kDecBuffers; ++u) {
        constexpr int kAhead = kDecBuffers - 1;
        issue(t0 + u + kAhead, kb[(u + kAhead) % kDecBuffers], vb[(u + kAhead) % kDecBuffers], kv[(u + kAhead) % kDecBuffers]);
        if (u == 0 || t0 + u < n_tiles) consume(kb[u], vb[u], kv[u]);  // uniform
        if (t0 + u == 0) DEC_STAMP_AFTER(2, acc[0][0]);  // first tile consumed (first K/V data arrived)
#ifdef UNIQUE_DEC_STAMPS
        if (t0 + u < n_tiles && t0 + u < kStampSlots - 6) DEC_STAMP_AFTER(6 + t0 + u, acc[0][0]);  // tile t0 + u consumed
        if (t0 + u == 0) {  // which compute unit this wave runs on (HW_ID: bits 8-11 CU, 13-15 SE; XCC_ID register)
          const int64_t sw_ = chunk_slot * kDecWaves + wave;
          if (lane == 0 && sw_ < kStampWaves)
            g_dec_stamps[sw_][5] = ((unsigned long long)__builtin_amdgcn_s_getreg((4 << 0) | (0 << 6) | (31 << 11)) << 32) |
                                   (unsigned)__builtin_amdgcn_s_getreg((20 << 0) | (0 << 6) | (3 << 11));
        }
#endif
      }
    }
  }

  DEC_STAMP_AFTER(3, acc[0][0]);  // streaming loop done
  // the wave's result: the sum of the lanes' l, and the output rows as they are (the parts are added below)
  l = rows_allreduce(l, OpSum());
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (4 * kg + i < kSlots) {
      float* dst = &sh.acc[wave][4 * kg + i][kt * kVB];
#pragma unroll
      for (int e = 0; e < kVB; e += 4)
        *reinterpret_cast<float4*>(dst + e) = make_float4(acc[e][i], acc[e + 1][i], acc[e + 2][i], acc[e + 3][i]);
    }
  }
  if (lane < G) { sh.m[wave][lane] = m; sh.l[wave][lane] = l; }
  __syncthreads();
  finish_chunk<bf16_t, D, G>(c, k, to, sh);
  DEC_STAMP(4);  // partial results stored
}

// Log-sum-exp merge of the chunk partials of one (sequence, query head) by kWaves waves; writes out (and lse). Lane s takes the (m, l)
// pair of chunk s, so the maximum, the per-chunk scales and the normaliser come from two wave reductions, in every wave for itself;
// wave w adds up the output rows of chunks w, w + kWaves, ... with the scale of chunk s broadcast from lane s, and the waves' sums
// are added through the LDS.
// What bounds it is the launch, 1.6 us in a chain of kernels, and round trips to what another kernel has just written. So the first
// 64 pairs and the first eight rows of every wave are requested at once, before anything is known of the row: `have` chunks are there to be
// read; the first ns_of() of them, whose loads are then on their way as well, hold results.
// A step us with a chain of the count, the pairs and eight rows of one wave after the other / so: 32K tokens, 32 chunks 19.7 / 18.2, a million
// tokens, 32 chunks 56.1 / 54.7, 96 rows of 5 chunks 61.9 / 61.2, 128 of 4 142.3 / 141.7.
template <int kWaves, int D>
struct MergeShared {
  float o[kWaves][D];
};
template <typename T, int D, int G, int kWaves, typename Chunks>
__device__ __forceinline__ void merge_chunks(const CacheView& c, int b, int h, int64_t base /*the row's first slot*/, int have, Chunks ns_of,
                                             const float* __restrict__ part_o, const float* __restrict__ part_ml,
                                             T* __restrict__ out, float* __restrict__ lse_out, MergeShared<kWaves, D>& sh) {
  constexpr int kPer = D / kWave;  // output elements per lane (1 or 2)
  constexpr int kBatch = 8;        // rows in flight per wave
  static_assert(kPer == 1 || kPer == 2, "head_dim 64 or 128");
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), g = h % G;
  const float2* ml = reinterpret_cast<const float2*>(part_ml) + base * G + g;  // (m, l) per (row, chunk, head)
  const float* po = part_o + (base * G + g) * D + lane * kPer;

  auto pair = [&](int s0) { return ml[(int64_t)min(s0 + lane, have - 1) * G]; };
  float2 v[kBatch];
  auto request = [&](int j0) {  // rows j0 + u * kWaves + wave; past the last chunk that chunk, whose scale is then zero
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const float* src = po + (int64_t)min(j0 + u * kWaves + wave, have - 1) * (G * D);
      if constexpr (kPer == 2) v[u] = *reinterpret_cast<const float2*>(src);
      else v[u] = make_float2(src[0], 0.f);
    }
  };
  const float2 first = have > 0 ? pair(0) : make_float2(kNegBig, 0.f);
  if (have > 0) request(0);
  const int ns = ns_of();

  float M = lane < ns ? first.x : kNegBig;
  for (int s0 = kWave; s0 < ns; s0 += kWave)
    if (s0 + lane < ns) M = fmaxf(M, pair(s0).x);
  M = group_allreduce<kWave>(M, OpMax());

  float L = 0.f, o[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) o[i] = 0.f;
  for (int s0 = 0; s0 < ns; s0 += kWave) {
    const float2 p = s0 == 0 ? first : pair(s0);
    const float sc = s0 + lane < ns ? fast_exp2(p.x - M) : 0.f;
    L = s0 + lane < ns ? fmaf(p.y, sc, L) : L;
    const int n = min(kWave, ns - s0);
    for (int j0 = 0; j0 < n; j0 += kBatch * kWaves) {
      if (s0 + j0 > 0) request(s0 + j0);
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int j = j0 + u * kWaves + wave;
        if (j >= n) break;  // uniform; a chunk without results may hold anything
        const float scj = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, sc), j));
        o[0] = fmaf(v[u].x, scj, o[0]);
        if constexpr (kPer == 2) o[1] = fmaf(v[u].y, scj, o[1]);
      }
    }
  }
  L = group_allreduce<kWave>(L, OpSum());
  const bool any = L > 0.f;
  T* dst = out + ((int64_t)b * c.H + h) * D + lane * kPer;
  if constexpr (kWaves > 1) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) sh.o[wave][lane * kPer + i] = o[i];
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int w = 1; w < kWaves; ++w)
#pragma unroll
      for (int i = 0; i < kPer; ++i) o[i] += sh.o[w][lane * kPer + i];
  }
#pragma unroll
  for (int i = 0; i < kPer; ++i) store_elem(dst + i, any ? o[i] / L : 0.f);
  if (lse_out && lane == 0) lse_out[(int64_t)b * c.H + h] = any ? (M + log2f(L)) * kLn2 : -INFINITY;
}

constexpr int kMergeWaves = 4;  // (eight: 18.3 and 55.0 us)
constexpr bool merge_alone(int chunks) { return chunks <= 8; }  // one wave

}  // namespace
}  // namespace unique
