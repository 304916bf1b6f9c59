// Paged decode attention over a list of logical pages per (sequence, KV head):
//   Eq. 5 of the paper when the list is the selected top-k set, Eq. 4 when it is every page.
//
// Split-K: the page list of a row is cut into chunks; one workgroup (4 waves) handles one chunk for all
// G query heads of the KV head at once, so every K/V byte is read exactly once per step. The work on a chunk
// is decode_core.hpp, which also has what is said of bf16 caches. fp32 caches: inside a wave
// each lane reads 16-byte chunks of K and V rows (a wave-wide load covers a contiguous 1 KiB of the
// page), the q.k dot products are reduced across the D/vec lanes that share a token with DPP row
// operations, and each group of lanes that shares a token row keeps its own online-softmax state, so
// the inner loop has no cross-row communication. States are merged (log-sum-exp) across lane groups,
// then across the 4 waves through LDS, and the chunk's partial (o, m, l) goes to the workspace; a
// second small kernel merges the chunks of a row and writes the output in the cache dtype (a row with
// a single chunk is written by the first kernel itself and the second is not launched). The merge stays a launch of its
// own: done by a row's last workgroup behind an agent-scope release and acquire it costs 8 us more than the launch
// (131K tokens, 128 rows), and with write-through stores instead of the release the step is no faster either.
// Logits are kept in the log2 domain (q is pre-multiplied by sm_scale * log2 e) so exp is one v_exp_f32.
#include <type_traits>

#include "decode_core.hpp"
#include "dense_plan.hpp"

namespace unique {
namespace {

template <typename T, int D, int S, int G, bool kNT>
__global__ __launch_bounds__(kDecWaves* kWave) void paged_decode_partial_kernel(
    CacheView c, const T* __restrict__ q, const int32_t* __restrict__ sel_pages,
    const int32_t* __restrict__ sel_count, int sel_stride, SplitPlan plan, float scale_log2,
    float* __restrict__ part_o, float* __restrict__ part_ml, T* __restrict__ out, float* __restrict__ lse_out) {
  __shared__ DecodeShared<T, D, G> sh;
  const int num_splits = plan.num_splits;
  int split, hkv, b;
  locate_chunk(c, plan, split, hkv, b);
  const int row = b * c.Hkv + hkv;
  const int64_t chunk_slot = (int64_t)row * num_splits + split;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;  // wave: scalar
  const int begin = split * plan.pages_per_split;
  DEC_STAMP(0);  // kernel entry
  // the first list entry of this lane is requested together with the lengths (row storage is sel_stride
  // entries long, so the load does not have to wait for the count)
  int first_lp = -1;
  {
    const int e = begin + wave + lane * kDecWaves;
    if (sel_pages && e < min(begin + plan.pages_per_split, sel_stride)) first_lp = sel_pages[(int64_t)row * sel_stride + e];
  }
  const int N = c.seq_lens[b];
  const int P = min((N + S - 1) / S, c.max_pages_hint);
  const int cnt = sel_pages ? min(sel_count[row], sel_stride) : P;
  const ChunkOut<T> to = {part_o, part_ml, out, lse_out, num_splits};
  if (begin >= cnt) {
    write_empty<T, D, G>(c, to, b, hkv);
    return;
  }
  const Chunk chunk = {hkv, b, begin, min(begin + plan.pages_per_split, cnt), N, chunk_slot};
  auto lookup = [&](int e, bool first, int& phys, int& ntok) {
    const int lp = !sel_pages ? e : (first ? first_lp : sel_pages[(int64_t)row * sel_stride + e]);
    if (lp >= 0 && lp < P) {
      const int ph = c.page_table[(int64_t)b * c.max_pages + lp];
      if (ph >= 0 && (int64_t)ph < c.num_phys) {
        phys = ph;
        ntok = min(S, N - lp * S);
      }
    }
  };
  decode_chunk<D, S, G, kNT>(c, q, chunk, wave, lane, lookup, scale_log2, to, sh);
}

template <typename T, int D, int G, int kWaves>
__global__ __launch_bounds__(kWaves* kWave) void paged_decode_merge_kernel(CacheView c, const int32_t* __restrict__ sel_count,
                                                                            int sel_stride, bool dense, int pages_per_split,
                                                                            int num_splits, const float* __restrict__ part_o,
                                                                            const float* __restrict__ part_ml,
                                                                            T* __restrict__ out, float* __restrict__ lse_out) {
  __shared__ MergeShared<kWaves, D> sh;
  const int h = blockIdx.x, b = blockIdx.y;
  const int row = b * c.Hkv + h / G;
  auto chunks = [&] {
    const int cnt = dense ? min((c.seq_lens[b] + c.S - 1) / c.S, c.max_pages_hint) : min(sel_count[row], sel_stride);
    return min(num_splits, (cnt + pages_per_split - 1) / pages_per_split);
  };
  merge_chunks<T, D, G, kWaves>(c, b, h, (int64_t)row * num_splits, num_splits, chunks, part_o, part_ml, out, lse_out, sh);
}

template <typename T, int D, int S, int G>
hipError_t launch_t(const CacheView& c, const void* q, const int32_t* sel, const int32_t* cnt, int sel_stride,
                    const SplitPlan& plan, bool stream_nt, float sm_scale, void* out, float* lse, float* partials, hipStream_t st) {
  float* part_ml = partials + (size_t)c.B * c.Hkv * plan.num_splits * G * D;
  auto go = [&](auto kernel) {
    const dim3 grid = plan.rotate ? dim3(c.Hkv, c.B, plan.num_splits) : dim3(plan.num_splits, c.Hkv, c.B);
    kernel<<<grid, dim3(kDecWaves * kWave), 0, st>>>(c, reinterpret_cast<const T*>(q), sel, cnt, sel_stride, plan,
                                                     decode_scale_log2(c, sm_scale), partials, part_ml, reinterpret_cast<T*>(out), lse);
  };
  if (stream_nt) go(paged_decode_partial_kernel<T, D, S, G, true>);
  else go(paged_decode_partial_kernel<T, D, S, G, false>);
  return hipGetLastError();
}

template <typename T, int D, int S>
hipError_t dispatch_g(const CacheView& c, const void* q, const int32_t* sel, const int32_t* cnt, int sel_stride,
                      const SplitPlan& plan, bool stream_nt, float sm_scale, void* out, float* lse, float* partials, hipStream_t st) {
  switch (c.H / c.Hkv) {
    case 1: return launch_t<T, D, S, 1>(c, q, sel, cnt, sel_stride, plan, stream_nt, sm_scale, out, lse, partials, st);
    case 2: return launch_t<T, D, S, 2>(c, q, sel, cnt, sel_stride, plan, stream_nt, sm_scale, out, lse, partials, st);
    case 4: return launch_t<T, D, S, 4>(c, q, sel, cnt, sel_stride, plan, stream_nt, sm_scale, out, lse, partials, st);
    case 8: return launch_t<T, D, S, 8>(c, q, sel, cnt, sel_stride, plan, stream_nt, sm_scale, out, lse, partials, st);
    default: return hipErrorInvalidValue;
  }
}

template <typename T, int D>
hipError_t dispatch_s(const CacheView& c, const void* q, const int32_t* sel, const int32_t* cnt, int sel_stride,
                      const SplitPlan& plan, bool stream_nt, float sm_scale, void* out, float* lse, float* partials, hipStream_t st) {
  switch (c.S) {
    case 8: return dispatch_g<T, D, 8>(c, q, sel, cnt, sel_stride, plan, stream_nt, sm_scale, out, lse, partials, st);
    case 16: return dispatch_g<T, D, 16>(c, q, sel, cnt, sel_stride, plan, stream_nt, sm_scale, out, lse, partials, st);
    case 32: return dispatch_g<T, D, 32>(c, q, sel, cnt, sel_stride, plan, stream_nt, sm_scale, out, lse, partials, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

#ifdef UNIQUE_DEC_STAMPS
extern "C" int unique_debug_dec_stamps(void** ptr, int* waves, int* slots) {
  *waves = kStampWaves;
  *slots = kStampSlots;
  return (int)hipGetSymbolAddress(ptr, HIP_SYMBOL(g_dec_stamps));
}

// Ceiling probe of the profiling build: the memory access of the sparse decode with everything else taken away.
// One wave fetches the 4 KiB K tile and the 4 KiB V tile of each of its (physical page, head) entries -- page ids
// straight from `list`, no page table, no arithmetic but an xor -- with kDepth tiles in flight. kPattern 0: every
// load instruction covers a contiguous 1 KiB; 1: K in the operand layout of the matrix-core q.k stage (64-byte
// pieces of 16 rows); 2: contiguous loads that go straight into LDS (second kernel below). Geometry as the decode kernel: rows x ceil(k / pages_per_wg) workgroups of `waves` waves.
namespace {
typedef unsigned int probe_u32x4 __attribute__((ext_vector_type(4)));
template <int kPattern, int kDepth>
__global__ __launch_bounds__(1024) void gather_probe_kernel(const char* __restrict__ kpool, const char* __restrict__ vpool,
                                                             const int32_t* __restrict__ list, int k, int pages_per_wg,
                                                             int waves, int heads, probe_u32x4* __restrict__ sink) {
  const int row = blockIdx.y, split = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int begin = split * pages_per_wg, end = min(begin + pages_per_wg, k);
  const int hkv = row % heads;
  const int n = min(kWave, (end - begin - wave + waves - 1) / waves);  // entries of this wave (lane i holds the i-th)
  int my_phys = 0;
  if (lane < n) my_phys = list[(size_t)row * k + begin + wave + lane * waves];
  probe_u32x4 acc = {0, 0, 0, 0};
  probe_u32x4 buf[kDepth][8];
  const int koff = kPattern == 0 ? lane * 16 : (lane % 16) * 256 + (lane / 16) * 16;
  const int kstep = kPattern == 0 ? 1024 : 64;
  auto issue = [&](int i, probe_u32x4(&b)[8]) {  // past the wave's last entry: its last page again (keeps the code straight-line)
    const int phys = __builtin_amdgcn_readlane(my_phys, max(min(i, n - 1), 0));
    const size_t base = ((size_t)phys * heads + hkv) * 4096;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      b[j] = __builtin_nontemporal_load(reinterpret_cast<const probe_u32x4*>(kpool + base + koff + j * kstep));
#pragma unroll
    for (int j = 0; j < 4; ++j)
      b[4 + j] = __builtin_nontemporal_load(reinterpret_cast<const probe_u32x4*>(vpool + base + lane * 16 + j * 1024));
  };
#pragma unroll
  for (int d = 0; d < kDepth; ++d) issue(d, buf[d]);
  for (int i = 0; i < n; i += kDepth) {
#pragma unroll
    for (int d = 0; d < kDepth; ++d) {
#pragma unroll
      for (int j = 0; j < 8; ++j) acc ^= buf[d][j];
      issue(i + d + kDepth, buf[d]);
    }
  }
  if (acc.x == 0x12345678u && acc.y == 0x9abcdef0u) sink[threadIdx.x] = acc;  // never true in practice; keeps the loads alive
}

// The same gather with the tiles sent straight into LDS (global_load_lds_dwordx4, no register between memory and
// LDS): a ring of kDepth tiles of 8 KiB per wave, each tile waited for with an explicit vmcnt and read back with
// ds_read_b128. Dynamic LDS: waves * kDepth * 8 KiB.
template <int kN>
__device__ __forceinline__ void probe_wait_vmcnt() {  // s_waitcnt vmcnt(kN) alone (expcnt and lgkmcnt fields left at their maximum)
  __builtin_amdgcn_s_waitcnt((kN & 0xF) | ((kN >> 4) << 14) | 0x0F70);
}
template <int kDepth>
__global__ __launch_bounds__(1024) void gather_probe_lds_kernel(const char* __restrict__ kpool,
                                                                 const char* __restrict__ vpool,
                                                                 const int32_t* __restrict__ list, int k, int pages_per_wg,
                                                                 int waves, int heads, probe_u32x4* __restrict__ sink) {
  extern __shared__ __attribute__((aligned(16))) char probe_lds[];
  typedef const __attribute__((address_space(1))) void* gptr_t;
  typedef __attribute__((address_space(3))) void* lptr_t;
  const int row = blockIdx.y, split = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int begin = split * pages_per_wg, end = min(begin + pages_per_wg, k);
  const int hkv = row % heads;
  const int n = min(kWave, (end - begin - wave + waves - 1) / waves);
  int my_phys = 0;
  if (lane < n) my_phys = list[(size_t)row * k + begin + wave + lane * waves];
  char* ring = probe_lds + (size_t)wave * kDepth * 8192;  // wave-uniform
  probe_u32x4 acc = {0, 0, 0, 0};
  auto issue = [&](int i, int d) {
    const int phys = __builtin_amdgcn_readlane(my_phys, max(min(i, n - 1), 0));
    const size_t base = ((size_t)phys * heads + hkv) * 4096 + lane * 16;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      __builtin_amdgcn_global_load_lds((gptr_t)(kpool + base + j * 1024), (lptr_t)(ring + d * 8192 + j * 1024), 16, 0, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      __builtin_amdgcn_global_load_lds((gptr_t)(vpool + base + j * 1024), (lptr_t)(ring + d * 8192 + 4096 + j * 1024), 16, 0, 0);
  };
#pragma unroll
  for (int d = 0; d < kDepth; ++d) issue(d, d);
  for (int i = 0; i < n; i += kDepth) {
#pragma unroll
    for (int d = 0; d < kDepth; ++d) {
      probe_wait_vmcnt<(kDepth - 1) * 8>();  // the oldest tile has landed; the younger ones may still be on their way
      asm volatile("" ::: "memory");
#pragma unroll
      for (int j = 0; j < 8; ++j) acc ^= *reinterpret_cast<const probe_u32x4*>(ring + d * 8192 + j * 1024 + lane * 16);
      asm volatile("" ::"v"(acc.x), "v"(acc.y), "v"(acc.z), "v"(acc.w) : "memory");  // the reads are done before the slot is refilled
      issue(i + d + kDepth, d);
    }
  }
  probe_wait_vmcnt<0>();
  if (acc.x == 0x12345678u && acc.y == 0x9abcdef0u) sink[threadIdx.x] = acc;
}
}  // namespace

// k_pool / v_pool: [num_pages][heads][4096 bytes]; list: int32 [rows][k] physical page ids (all < num_pages, which the
// caller guarantees); sink: 16 KiB of device memory. Returns a hipError_t.
extern "C" int unique_debug_gather_probe(const void* k_pool, const void* v_pool, const int32_t* list, int rows, int k,
                                         int heads, int pages_per_wg, int waves, int depth, int pattern, void* sink,
                                         void* stream) {
  if (rows < 1 || k < 1 || heads < 1 || waves < 1 || waves > 16 || pages_per_wg < waves || pages_per_wg > 64 * waves)
    return (int)hipErrorInvalidValue;
  const dim3 grid((k + pages_per_wg - 1) / pages_per_wg, rows), block(waves * kWave);
  auto go = [&](auto kernel) {
    kernel<<<grid, block, 0, (hipStream_t)stream>>>((const char*)k_pool, (const char*)v_pool, list, k, pages_per_wg,
                                                    waves, heads, (probe_u32x4*)sink);
  };
  if (pattern == 2) {  // through LDS
    const size_t lds = (size_t)waves * depth * 8192;
    if (lds > 160 * 1024 || (depth != 2 && depth != 4)) return (int)hipErrorInvalidValue;
    auto go_lds = [&](auto kernel) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return (int)e;
      kernel<<<grid, block, lds, (hipStream_t)stream>>>((const char*)k_pool, (const char*)v_pool, list, k, pages_per_wg,
                                                        waves, heads, (probe_u32x4*)sink);
      return (int)hipGetLastError();
    };
    return depth == 2 ? go_lds(gather_probe_lds_kernel<2>) : go_lds(gather_probe_lds_kernel<4>);
  }
  if (pattern == 0 && depth == 2) go(gather_probe_kernel<0, 2>);
  else if (pattern == 0 && depth == 4) go(gather_probe_kernel<0, 4>);
  else if (pattern == 1 && depth == 2) go(gather_probe_kernel<1, 2>);
  else if (pattern == 1 && depth == 4) go(gather_probe_kernel<1, 4>);
  else return (int)hipErrorInvalidValue;
  return (int)hipGetLastError();
}
#endif

bool decode_supported(int dtype, int D, int S, int G) {
  return (dtype == 0 || dtype == 1) && (D == 64 || D == 128) && (S == 8 || S == 16 || S == 32) &&
         (G == 1 || G == 2 || G == 4 || G == 8);
}

SplitPlan selection_plan(const CacheView& c, int top_k) {
  const int elem = c.dtype == 0 ? 4 : 2;
  return plan_splits(c.B, c.Hkv, top_k, c.max_pages_hint, c.S * c.D * 2 * elem, elem == 4 && c.H == 8 * c.Hkv);
}

size_t plan_partial_floats(const CacheView& c, const SplitPlan& plan) {
  return (size_t)c.B * c.Hkv * plan.num_splits * (size_t)(c.H / c.Hkv) * (size_t)(c.D + 2);
}

size_t decode_partial_floats(const CacheView& c, int max_list_len) {
  return plan_partial_floats(c, most_splits(c.B * c.Hkv, max_list_len));
}

bool decode_streams(const CacheView& c, int max_list_len) {
  return (int64_t)c.B * c.Hkv * max_list_len * c.S * c.D * 2 * (c.dtype == 0 ? 4 : 2) > kStreamNtBytes;
}

float decode_scale_log2(const CacheView& c, float sm_scale) {
  return (sm_scale > 0.f ? sm_scale : 1.0f / sqrtf((float)c.D)) * kLog2e;
}

hipError_t launch_merge(const CacheView& c, const int32_t* d_sel_count, int sel_stride, const SplitPlan& plan, float* d_partials,
                        void* d_out, float* d_lse_out, hipStream_t stream) {
  auto with = [&](auto elem, auto dim, auto group) {
    using T = decltype(elem);
    constexpr int D = decltype(dim)::value, G = decltype(group)::value;
    const float* part_ml = d_partials + (size_t)c.B * c.Hkv * plan.num_splits * G * D;
    auto go = [&](auto kernel, int waves) {
      kernel<<<dim3(c.H, c.B), dim3(waves * kWave), 0, stream>>>(c, d_sel_count, sel_stride, d_sel_count == nullptr, plan.pages_per_split,
                                                                 plan.num_splits, d_partials, part_ml, reinterpret_cast<T*>(d_out), d_lse_out);
      return hipGetLastError();
    };
    return merge_alone(plan.num_splits) ? go(paged_decode_merge_kernel<T, D, G, 1>, 1)
                                        : go(paged_decode_merge_kernel<T, D, G, kMergeWaves>, kMergeWaves);
  };
  auto with_group = [&](auto elem, auto dim) {
    switch (c.H / c.Hkv) {
      case 1: return with(elem, dim, std::integral_constant<int, 1>());
      case 2: return with(elem, dim, std::integral_constant<int, 2>());
      case 4: return with(elem, dim, std::integral_constant<int, 4>());
      case 8: return with(elem, dim, std::integral_constant<int, 8>());
      default: return hipErrorInvalidValue;
    }
  };
  auto with_dim = [&](auto elem) {
    return c.D == 64 ? with_group(elem, std::integral_constant<int, 64>()) : with_group(elem, std::integral_constant<int, 128>());
  };
  return c.dtype == 0 ? with_dim(float()) : with_dim(bf16_t());
}

hipError_t launch_decode(const CacheView& c, const void* d_q, const int32_t* d_sel_pages,
                         const int32_t* d_sel_count, int sel_stride, int max_list_len, float sm_scale,
                         void* d_out, float* d_lse_out, float* d_partials, hipStream_t stream) {
  if (!d_sel_pages && dense_balances(c.B, c.Hkv, c.max_pages_hint, c.S * c.D * 2 * (c.dtype == 0 ? 4 : 2))) {
    auto run = [&](auto launch) { return launch(c, d_q, sm_scale, d_out, d_lse_out, d_partials, stream); };
    return c.dtype == 0 ? (c.D == 64 ? run(launch_dense<float, 64>) : run(launch_dense<float, 128>))
                        : (c.D == 64 ? run(launch_dense<bf16_t, 64>) : run(launch_dense<bf16_t, 128>));
  }
  const SplitPlan plan = d_sel_pages ? selection_plan(c, max_list_len) : most_splits(c.B * c.Hkv, max_list_len);
  const bool nt = decode_streams(c, max_list_len);
  auto go = [&](auto dispatch) {
    return dispatch(c, d_q, d_sel_pages, d_sel_count, sel_stride, plan, nt, sm_scale, d_out, d_lse_out, d_partials, stream);
  };
  const hipError_t e = c.dtype == 0 ? (c.D == 64 ? go(dispatch_s<float, 64>) : go(dispatch_s<float, 128>))
                                    : (c.D == 64 ? go(dispatch_s<bf16_t, 64>) : go(dispatch_s<bf16_t, 128>));
  if (e != hipSuccess || plan.num_splits == 1) return e;  // one chunk per row: the partial kernel wrote the output
  return launch_merge(c, d_sel_pages ? d_sel_count : nullptr, sel_stride, plan, d_partials, d_out, d_lse_out, stream);
}

}  // namespace unique
