// Dense decode of batches whose sequences may differ in length: chunks of nearly equal size from the lengths on the device.
//
// The host knows only the longest sequence, so most_splits cuts every row at the same multiples of 256 pages, and a ragged batch
// leaves some compute units with two full chunks and others with one: 8 sequences of 2000 to 60000 tokens read 811 MB in 142 us,
// 5.7 TB/s, where an even batch reaches 6.7. Here every workgroup adds up the pages of the batch, finds the smallest
// chunk with which the chunks fit the workgroups that run at the same time (or a multiple of them), cuts every row into
// equal chunks not longer than that, and takes the chunk of its index. That batch now takes 128 us, 6.3 TB/s; 32 sequences of 4K
// to 131K tokens (5.7 GB) 1832 before, 911 now. Other sizes: dense_plan.hpp.
#include <type_traits>

#include "decode_core.hpp"
#include "dense_plan.hpp"

namespace unique {
namespace {

// The chunks of a batch, the same in every wave that asks: lane b holds those of sequence b.
struct BatchChunks {
  int len;     // tokens of sequence `lane`
  int pages;
  int chunks;  // per row of that sequence
  int before;  // chunks per head of the sequences before it
};

__device__ __forceinline__ int wave_sum(int x) { return __builtin_amdgcn_readlane(wave_inclusive_scan(x), kWave - 1); }

// false: no chunk has the index w, or a larger one
__device__ __forceinline__ bool cut_batch(const CacheView& c, int S, int max_chunks, int w, BatchChunks& bc) {
  const int lane = threadIdx.x % kWave;
  bc.len = lane < c.B ? c.seq_lens[lane] : 0;
  bc.pages = max(0, min((bc.len + S - 1) / S, c.max_pages_hint));
  const int rows = c.B * c.Hkv;
  const int total = wave_sum(bc.pages) * c.Hkv, slots = dense_slots(total, max_chunks);
  const bool room = dense_has_room(rows, slots, max_chunks);
  if (w >= (room ? slots + rows : slots)) return false;  // most workgroups of a launch whose bound is far above the lengths
  if (__ballot(lane < c.B && bc.pages != __builtin_amdgcn_readfirstlane(bc.pages)) == 0) {
    bc.chunks = lane < c.B ? dense_even_chunks(bc.pages, rows, slots) : 0;
  } else {
    bc.chunks = dense_row_chunks(bc.pages, dense_rate(total, rows, slots, [&](uint32_t rate) {
      return wave_sum(dense_row_weight(bc.pages, rate, room)) * c.Hkv;
    }));
  }
  bc.before = wave_inclusive_scan(bc.chunks) - bc.chunks;
  return true;
}

template <typename T, int D, int S, int G, bool kNT>
__global__ __launch_bounds__(kDecWaves* kWave) void paged_decode_dense_kernel(CacheView c, const T* __restrict__ q, int max_chunks,
                                                                              float scale_log2, float* __restrict__ part_o,
                                                                              float* __restrict__ part_ml) {
  __shared__ DecodeShared<T, D, G> sh;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;  // wave: scalar
  const int w = blockIdx.x;
  BatchChunks bc;
  if (!cut_batch(c, S, max_chunks, w, bc)) return;
  const unsigned long long here = __ballot(w >= bc.before * c.Hkv && w < (bc.before + bc.chunks) * c.Hkv);
  if (here == 0) return;  // beyond the last chunk
  const int b = __ffsll(here) - 1;
  const int P = __builtin_amdgcn_readlane(bc.pages, b), n = __builtin_amdgcn_readlane(bc.chunks, b);
  const int i = w - __builtin_amdgcn_readlane(bc.before, b) * c.Hkv;  // chunk `split` of head hkv
  const int hkv = i / n, split = i % n, len = (P + n - 1) / n;
  const int begin = split * len, end = min(begin + len, P);
  const int N = __builtin_amdgcn_readlane(bc.len, b);
  const ChunkOut<T> to = {part_o, part_ml, nullptr, nullptr, 2};
  const Chunk chunk = {hkv, b, begin, max(begin, end), N, w};
  auto lookup = [&](int e, bool, int& phys, int& ntok) {
    const int ph = c.page_table[(int64_t)b * c.max_pages + e];
    if (ph >= 0 && (int64_t)ph < c.num_phys) {
      phys = ph;
      ntok = min(S, N - e * S);
    }
  };
  decode_chunk<D, S, G, kNT>(c, q, chunk, wave, lane, lookup, scale_log2, to, sh);
}

template <typename T, int D, int G, int kWaves>
__global__ __launch_bounds__(kWaves* kWave) void paged_decode_dense_merge_kernel(CacheView c, int max_chunks,
                                                                                  const float* __restrict__ part_o,
                                                                                  const float* __restrict__ part_ml, T* __restrict__ out,
                                                                                  float* __restrict__ lse_out) {
  __shared__ MergeShared<kWaves, D> sh;
  const int h = blockIdx.x, b = blockIdx.y, hkv = h / G;
  BatchChunks bc;
  cut_batch(c, c.S, max_chunks, 0, bc);
  const int n = __builtin_amdgcn_readlane(bc.chunks, b);
  const int64_t base = (int64_t)__builtin_amdgcn_readlane(bc.before, b) * c.Hkv + (int64_t)hkv * n;
  merge_chunks<T, D, G, kWaves>(c, b, h, base, n, [&] { return n; }, part_o, part_ml, out, lse_out, sh);
}

template <typename T, int D, int S, int G>
hipError_t launch_t(const CacheView& c, const void* q, float sm_scale, void* out, float* lse, float* partials, hipStream_t st) {
  const int max_chunks = dense_max_chunks(c.B * c.Hkv, c.max_pages_hint);
  float* part_ml = partials + (size_t)max_chunks * G * D;
  auto go = [&](auto kernel) {
    kernel<<<dim3(max_chunks), dim3(kDecWaves * kWave), 0, st>>>(c, reinterpret_cast<const T*>(q), max_chunks,
                                                                 decode_scale_log2(c, sm_scale), partials, part_ml);
  };
  if (decode_streams(c, c.max_pages_hint)) go(paged_decode_dense_kernel<T, D, S, G, true>);
  else go(paged_decode_dense_kernel<T, D, S, G, false>);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  auto merge = [&](auto kernel, int waves) {
    kernel<<<dim3(c.H, c.B), dim3(waves * kWave), 0, st>>>(c, max_chunks, partials, part_ml, reinterpret_cast<T*>(out), lse);
    return hipGetLastError();
  };
  return dense_merge_alone(c.B * c.Hkv) ? merge(paged_decode_dense_merge_kernel<T, D, G, 1>, 1)
                                        : merge(paged_decode_dense_merge_kernel<T, D, G, kMergeWaves>, kMergeWaves);
}

template <typename T, int D, int S>
hipError_t dispatch_g(const CacheView& c, const void* q, float sm_scale, void* out, float* lse, float* partials, hipStream_t st) {
  switch (c.H / c.Hkv) {
    case 1: return launch_t<T, D, S, 1>(c, q, sm_scale, out, lse, partials, st);
    case 2: return launch_t<T, D, S, 2>(c, q, sm_scale, out, lse, partials, st);
    case 4: return launch_t<T, D, S, 4>(c, q, sm_scale, out, lse, partials, st);
    case 8: return launch_t<T, D, S, 8>(c, q, sm_scale, out, lse, partials, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// One translation unit per element type and head dimension: UNIQUE_ELEM, UNIQUE_DIM.
template <>
hipError_t launch_dense<UNIQUE_ELEM, UNIQUE_DIM>(const CacheView& c, const void* d_q, float sm_scale, void* d_out, float* d_lse_out,
                                                 float* d_partials, hipStream_t st) {
  switch (c.S) {
    case 8: return dispatch_g<UNIQUE_ELEM, UNIQUE_DIM, 8>(c, d_q, sm_scale, d_out, d_lse_out, d_partials, st);
    case 16: return dispatch_g<UNIQUE_ELEM, UNIQUE_DIM, 16>(c, d_q, sm_scale, d_out, d_lse_out, d_partials, st);
    case 32: return dispatch_g<UNIQUE_ELEM, UNIQUE_DIM, 32>(c, d_q, sm_scale, d_out, d_lse_out, d_partials, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace unique
