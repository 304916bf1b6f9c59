// Device code of the page score that the score kernel (score.hip) and the kernel of a whole small step (step.hip) share: the score
// of one (page, KV head) mean row by 8 lanes, and the statistics of a page that has received a token.
#pragma once
#include "device_utils.hpp"
#include "kernels.hpp"

namespace unique {
namespace {

constexpr int kRowLanes = 8;                   // lanes per (page, head) row
constexpr int kRowsPerWave = kWave / kRowLanes;
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// kE consecutive query elements, loaded as raw 32-bit words, as floats (kE = 4 or 8)
template <int kE>
__device__ __forceinline__ void unpack_q(const uint32_t (&w)[kE], float (&out)[kE], const float*) {
#pragma unroll
  for (int i = 0; i < kE; ++i) out[i] = bits_to_float(w[i]);
}
template <int kE>
__device__ __forceinline__ void unpack_q(const uint32_t (&w)[kE / 2], float (&out)[kE], const bf16_t*) {
#pragma unroll
  for (int i = 0; i < kE / 2; ++i) {
    out[2 * i] = bits_to_float(w[i] << 16);
    out[2 * i + 1] = bits_to_float(w[i] & 0xffff0000u);
  }
}

// The G queries of a KV head as a lane of a row needs them, and the score of a row with them.
// T: element type of q; TS: element type of the stored means (float, or bf16_t for bf16 statistics).
template <typename T, typename TS, int D, int G>
struct RowScorer {
  static constexpr int kE = Elem<TS>::kVec;                  // mean elements per 16-byte load
  static constexpr int kChunks = D / (kE * kRowLanes);       // 16-byte loads per lane per row
  static constexpr int kQWords = kE * (int)sizeof(T) / 4;    // raw query words per chunk
  // bf16 queries against bf16 means: packed bf16 pairs go straight into v_dot2_f32_bf16 (two products
  // per instruction accumulated in fp32, no unpacking); every other combination multiplies in fp32.
  static constexpr bool kDot2 = sizeof(T) == 2 && sizeof(TS) == 2;
  uint32_t qraw[G][kChunks][kQWords];
  float qv[kDot2 ? 1 : G][kChunks][kE];
  uint32_t qp[kDot2 ? G : 1][kChunks][kE / 2];
  float off[G];

  // q: the first query of the group; cl: the lane's place in its row
  __device__ __forceinline__ void request(const T* q, int cl) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
#pragma unroll
      for (int j = 0; j < kChunks; ++j) {
        const uint32_t* qsrc = reinterpret_cast<const uint32_t*>(q + g * D + j * (kE * kRowLanes) + cl * kE);
        if constexpr (kQWords == 2) {
          const uint2 v = *reinterpret_cast<const uint2*>(qsrc);
          qraw[g][j][0] = v.x; qraw[g][j][1] = v.y;
        } else {
#pragma unroll
          for (int w = 0; w < kQWords; w += 4) {
            const uint4 v = *reinterpret_cast<const uint4*>(qsrc + w);
            qraw[g][j][w] = v.x; qraw[g][j][w + 1] = v.y; qraw[g][j][w + 2] = v.z; qraw[g][j][w + 3] = v.w;
          }
        }
      }
    }
  }

  __device__ __forceinline__ void unpack(float lambda) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float qq = 0.f;
#pragma unroll
      for (int j = 0; j < kChunks; ++j) {
        float qf[kE];
        unpack_q<kE>(qraw[g][j], qf, (const T*)nullptr);
#pragma unroll
        for (int i = 0; i < kE; ++i) qq = fmaf(qf[i], qf[i], qq);
        if constexpr (kDot2) {
#pragma unroll
          for (int i = 0; i < kE / 2; ++i) qp[g][j][i] = qraw[g][j][i];
        } else {
#pragma unroll
          for (int i = 0; i < kE; ++i) qv[g][j][i] = qf[i];
        }
      }
      qq = group_allreduce<kRowLanes>(qq, OpSum());
      off[g] = lambda * sqrtf(qq);
    }
  }

  // every lane of the row gets the score of the row's mean `mc` and std `sd`
  __device__ __forceinline__ float score(const Raw16 (&mc)[kChunks], float sd) const {
    float mf[kDot2 ? 1 : kChunks][kE];
    if constexpr (!kDot2) {
#pragma unroll
      for (int j = 0; j < kChunks; ++j) unpack_raw(mc[j], mf[j], (const TS*)nullptr);
    }
    float best = 0.f;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float dot = 0.f;
      if constexpr (kDot2) {
#pragma unroll
        for (int j = 0; j < kChunks; ++j) {
          const uint32_t mw[4] = {mc[j].v.x, mc[j].v.y, mc[j].v.z, mc[j].v.w};
#pragma unroll
          for (int i = 0; i < 4; ++i)
            dot = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, qp[g][j][i]),
                                                  __builtin_bit_cast(bf16x2_t, mw[i]), dot, false);
        }
      } else {
#pragma unroll
        for (int j = 0; j < kChunks; ++j)
#pragma unroll
          for (int i = 0; i < kE; ++i) dot = fmaf(qv[g][j][i], mf[j][i], dot);
      }
      dot = group_allreduce<kRowLanes>(dot, OpSum());
      const float sc = fmaf(off[g], sd, dot);
      best = (g == 0) ? sc : fmaxf(best, sc);
    }
    return best;
  }
};

// Statistics of the last (possibly partial) page of a sequence for one KV head, recomputed from the page's n keys by a wave. The
// lane layout, the order of every sum and the cross-lane reductions are those of the bulk statistics kernel, so the record is
// bit-identical to what unique_update_page_stats writes. Pages of up to kMaxTokens tokens; the loads are predicated.
template <typename T, int D, int kMaxTokens>
struct PageRefresh {
  static constexpr int kVec = Elem<T>::kVec;
  static constexpr int kLanesPerTok = D / kVec;
  static constexpr int kTokPerLoad = kWave / kLanesPerTok;
  static constexpr int kMaxLoads = kMaxTokens / kTokPerLoad;
  // the page is read once and kept as raw 16-byte chunks; both passes unpack from registers
  Raw16 raw[kMaxLoads];
  float mean[kVec], std;  // every lane: the channels of its place in a token; the page's std

  __device__ __forceinline__ void request(const T* keys, int n, int lane) {
    const int tr = lane / kLanesPerTok;
    const T* base = keys + lane % kLanesPerTok * kVec;
#pragma unroll
    for (int j = 0; j < kMaxLoads; ++j) {
      const int tok = j * kTokPerLoad + tr;
      raw[j] = tok < n ? load_raw(base + (int64_t)tok * D) : zero_raw();
    }
  }

  __device__ __forceinline__ void reduce(int n, int lane) {
    const int tr = lane / kLanesPerTok;
    const float inv_n = 1.0f / (float)n;
    float sum[kVec];
#pragma unroll
    for (int i = 0; i < kVec; ++i) sum[i] = 0.f;
#pragma unroll
    for (int j = 0; j < kMaxLoads; ++j) {
      if (j * kTokPerLoad + tr < n) {
        float x[kVec];
        unpack_raw(raw[j], x, (const T*)nullptr);
#pragma unroll
        for (int i = 0; i < kVec; ++i) sum[i] += x[i];
      }
    }
#pragma unroll
    for (int i = 0; i < kVec; ++i) mean[i] = cross_group_allreduce<kLanesPerTok>(sum[i], OpSum()) * inv_n;
    float ss = 0.f;
#pragma unroll
    for (int j = 0; j < kMaxLoads; ++j) {
      if (j * kTokPerLoad + tr < n) {
        float x[kVec];
        unpack_raw(raw[j], x, (const T*)nullptr);
#pragma unroll
        for (int i = 0; i < kVec; ++i) {
          const float dev = x[i] - mean[i];
          ss = fmaf(dev, dev, ss);  // explicit: all statistics paths must round identically
        }
      }
    }
    ss = group_allreduce<kWave>(ss, OpSum());
    std = sqrtf(ss * inv_n);
  }

  // the mean row at `row`, as fp32 or bf16 (16-byte aligned)
  __device__ __forceinline__ void store_mean(void* row, bool bf16, int lane) const {
    if (lane / kLanesPerTok != 0) return;
    const int at = lane * kVec;
    if (bf16) {
      bf16_t* m = reinterpret_cast<bf16_t*>(row) + at;
      uint32_t w[kVec / 2];
#pragma unroll
      for (int i = 0; i < kVec; i += 2)
        w[i / 2] = (uint32_t)float_to_bf16(mean[i]) | ((uint32_t)float_to_bf16(mean[i + 1]) << 16);
      if constexpr (kVec == 8) *reinterpret_cast<uint4*>(m) = make_uint4(w[0], w[1], w[2], w[3]);
      else *reinterpret_cast<uint2*>(m) = make_uint2(w[0], w[1]);
    } else {
      float* m = reinterpret_cast<float*>(row) + at;
#pragma unroll
      for (int i = 0; i < kVec; i += 4)
        *reinterpret_cast<float4*>(m + i) = make_float4(mean[i], mean[i + 1], mean[i + 2], mean[i + 3]);
    }
  }
};

}  // namespace
}  // namespace unique
