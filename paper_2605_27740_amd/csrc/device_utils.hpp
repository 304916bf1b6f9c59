// Device-side helpers shared by the gfx950 kernels: 16-byte vector loads of fp32 / bf16 rows,
// bf16 <-> fp32 conversion, and cross-lane reductions over groups of 8..64 lanes (wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace unique {

using bf16_t = uint16_t;  // raw bf16 bit pattern

constexpr int kWave = 64;

template <typename T> struct Elem;
template <> struct Elem<float> { static constexpr int kVec = 4; };   // elements per 16-byte load
template <> struct Elem<bf16_t> { static constexpr int kVec = 8; };

__device__ __forceinline__ float bits_to_float(uint32_t u) { return __uint_as_float(u); }

// fp32 -> bf16, round to nearest even; NaN stays NaN.
__device__ __forceinline__ bf16_t float_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)((u >> 16) | 0x0040u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

__device__ __forceinline__ void store_elem(float* p, float v) { *p = v; }
__device__ __forceinline__ void store_elem(bf16_t* p, float v) { *p = float_to_bf16(v); }
__device__ __forceinline__ float load_elem(const float* p) { return *p; }
__device__ __forceinline__ float load_elem(const bf16_t* p) { return bits_to_float((uint32_t)(*p) << 16); }

// One 16-byte load expanded to fp32 lanes. p must be 16-byte aligned.
__device__ __forceinline__ void load_vec(const float* p, float (&out)[4]) {
  const float4 v = *reinterpret_cast<const float4*>(p);
  out[0] = v.x; out[1] = v.y; out[2] = v.z; out[3] = v.w;
}
__device__ __forceinline__ void unpack_bf16x8(const uint4& v, float (&out)[8]) {
  out[0] = bits_to_float(v.x << 16); out[1] = bits_to_float(v.x & 0xffff0000u);
  out[2] = bits_to_float(v.y << 16); out[3] = bits_to_float(v.y & 0xffff0000u);
  out[4] = bits_to_float(v.z << 16); out[5] = bits_to_float(v.z & 0xffff0000u);
  out[6] = bits_to_float(v.w << 16); out[7] = bits_to_float(v.w & 0xffff0000u);
}
__device__ __forceinline__ void load_vec(const bf16_t* p, float (&out)[8]) {
  const uint4 v = *reinterpret_cast<const uint4*>(p);
  unpack_bf16x8(v, out);
}

// Raw 16-byte register image of a row chunk, so that loads can be issued early and unpacked late.
struct Raw16 { uint4 v; };
__device__ __forceinline__ Raw16 load_raw(const void* p) {
  Raw16 r; r.v = *reinterpret_cast<const uint4*>(p); return r;
}
// The same load marked non-temporal: for data that is read once per launch (K/V pages, statistic
// records). A plain streaming read measures about 6.3 TB/s on MI355X, a non-temporal one about 7.1 TB/s.
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
// `nt` is uniform per launch: small working sets are better left to the caches (they are re-read by the next step).
__device__ __forceinline__ Raw16 load_raw_stream(const void* p, bool nt) {
  if (nt) {
    const u32x4_t t = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
    Raw16 r; r.v = make_uint4(t.x, t.y, t.z, t.w); return r;
  }
  return load_raw(p);
}
__device__ __forceinline__ Raw16 zero_raw() { Raw16 r; r.v = make_uint4(0u, 0u, 0u, 0u); return r; }
__device__ __forceinline__ void unpack_raw(const Raw16& r, float (&out)[4], const float*) {
  out[0] = bits_to_float(r.v.x); out[1] = bits_to_float(r.v.y);
  out[2] = bits_to_float(r.v.z); out[3] = bits_to_float(r.v.w);
}
__device__ __forceinline__ void unpack_raw(const Raw16& r, float (&out)[8], const bf16_t*) {
  unpack_bf16x8(r.v, out);
}

// ---- DPP lane exchange inside a row of 16 lanes (no LDS traffic) ----
template <int kCtrl>
__device__ __forceinline__ float dpp_mov(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kCtrl, 0xf, 0xf, true));
}
constexpr int kDppXor1 = 0xB1;        // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;        // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141; // lane i <-> 7-i inside each 8
constexpr int kDppMirror = 0x140;     // lane i <-> 15-i inside each 16
constexpr int kDppRor8 = 0x128;       // lane i <-> i^8 inside each 16

// Minimum / maximum of an unsigned value over the 64 lanes of a wave (every lane gets the result): four DPP
// exchanges inside the rows of 16 lanes, then two swaps between rows (a shuffle through the LDS takes 100 cycles more).
template <bool kMax>
__device__ __forceinline__ uint32_t wave_allreduce_minmax(uint32_t x) {
  auto op = [](uint32_t a, uint32_t b) { return kMax ? (a > b ? a : b) : (a < b ? a : b); };
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kDppXor1, 0xf, 0xf, true));
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kDppXor2, 0xf, 0xf, true));
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kDppHalfMirror, 0xf, 0xf, true));
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kDppMirror, 0xf, 0xf, true));
  auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  x = op(r[0], r[1]);
  r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return op(r[0], r[1]);
}

// Inclusive prefix sum over the 64 lanes of a wave: four row shifts inside each row of 16 lanes (a lane whose
// source lies outside its row adds 0), then lane 15 of rows 0 and 2 is added to rows 1 and 3, then lane 31 to
// rows 2 and 3. No LDS traffic.
__device__ __forceinline__ int wave_inclusive_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);   // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);   // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);   // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);   // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
  return x;
}

// Order-preserving map of fp32 to uint32 (a larger score has a larger key; -0 and +0 are equal). A NaN becomes 1, below
// -inf, and 0 means "no page".
__device__ __forceinline__ uint32_t score_key(float f) {
  const uint32_t u = __float_as_uint(f + 0.f);  // -0 becomes +0
  const uint32_t k = u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
  return f != f ? 1u : k;
}

struct OpSum { __device__ __forceinline__ float operator()(float a, float b) const { return a + b; } };
struct OpMax { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };

// A value combined with that of the lane 16 or 32 away, by a swap of rows of 16 lanes between two copies of it; op commutes.
template <typename Op>
__device__ __forceinline__ float with_lane_xor16(float x, Op op) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <typename Op>
__device__ __forceinline__ float with_lane_xor32(float x, Op op) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// All-reduce over aligned groups of kWidth consecutive lanes (kWidth in 1,2,4,8,16,32,64): every lane
// of a group ends with the group's result. kLds: lanes 16 and 32 apart exchange through the LDS, which takes longer for one value but
// leaves the vector ALUs to others: the statistics kernel, 2048 tokens of each of 4 sequences, 5.44 us with row swaps, 5.15 so; the attention of eight
// heads over an fp32 cache 4 % (decode_core.hpp).
template <int kWidth, bool kLds = false, typename Op>
__device__ __forceinline__ float group_allreduce(float x, Op op) {
  static_assert(kWidth == 1 || kWidth == 2 || kWidth == 4 || kWidth == 8 || kWidth == 16 || kWidth == 32 ||
                kWidth == 64, "group width");
  if constexpr (kWidth >= 2) x = op(x, dpp_mov<kDppXor1>(x));
  if constexpr (kWidth >= 4) x = op(x, dpp_mov<kDppXor2>(x));
  if constexpr (kWidth >= 8) x = op(x, dpp_mov<kDppHalfMirror>(x));
  if constexpr (kWidth >= 16) x = op(x, dpp_mov<kDppMirror>(x));
  if constexpr (kWidth >= 32) x = kLds ? op(x, __shfl_xor(x, 16, kWave)) : with_lane_xor16(x, op);
  if constexpr (kWidth >= 64) x = kLds ? op(x, __shfl_xor(x, 32, kWave)) : with_lane_xor32(x, op);
  return x;
}

// All-reduce across the kGroups = 64 / kStride lane groups of a wave: combines lanes that share
// lane % kStride. kStride in {8, 16, 32, 64}. kLds as above, and for lanes 8 apart.
template <int kStride, bool kLds = false, typename Op>
__device__ __forceinline__ float cross_group_allreduce(float x, Op op) {
  if constexpr (kStride <= 8) x = kLds ? op(x, __shfl_xor(x, 8, kWave)) : op(x, dpp_mov<kDppRor8>(x));
  if constexpr (kStride <= 16) x = kLds ? op(x, __shfl_xor(x, 16, kWave)) : with_lane_xor16(x, op);
  if constexpr (kStride <= 32) x = kLds ? op(x, __shfl_xor(x, 32, kWave)) : with_lane_xor32(x, op);
  return x;
}

}  // namespace unique
