// KV append for gfx950: the decode step's new K and V rows go into their slot
// of the paged pools before attention runs (paper Section II-A: the KV cache is
// updated with each newly generated token).  A few hundred KiB per call, so latency is all there
// is: the launch itself (1.65 us for an empty kernel between two others), then length -> table entry ->
// slot.  A workgroup has one request, K's chunks of 16 bytes and then V's, a lane each: the two look-ups
// are scalar, nothing is divided, and the new rows are asked for before the length is known.  Against a chunk of both pools per
// lane of a flat grid, 64-bit divisions by the row and rows loaded last, us from one launch to the next on tables and slots that
// are warm: one request on 8 KV heads 2.95 -> 2.81, 64 3.19 -> 3.01, 64 on 8-bit pools 3.64 -> 3.06, 1000 at D = 256 4.88 -> 4.36;
// with the attention behind it one request of 8191 tokens 18.5 -> 18.2, 64 of 64 on 8-bit pools 13.4 -> 12.9.  Behind a long
// kernel that has read the pools, 24 requests and more take 4.6 to 5 us either way.
#include "pkv_kernels.h"

namespace pkv {
namespace {

constexpr int kAppendThreads = 256;

// Where the row of a new token goes.
struct AppendTarget {
  const int32_t* block_tables;
  const int32_t* context_lens;
  int32_t* id_faults;
  int row_chunks;      // 16-byte chunks of a request's new K (or V) rows: Hkv * D / 8
  int log_chunks;      // log2 of those of one KV head, D / 8
  int log_block;       // log2 of the block size
  int MAXB, Hkv, max_ctx, NB;
};

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float to_range(float y) {
  return (y != y) ? y : fminf(fmaxf(y, -448.f), 448.f);   // NaN stays NaN
}
// two bf16 of one dword, scaled -> two e4m3 bytes in the chosen half of `old`
template <bool kHigh>
__device__ __forceinline__ int quantise2(uint32_t pair, float scale, int old) {
  const float a = __uint_as_float(pair << 16) / scale;
  const float b = __uint_as_float(pair & 0xffff0000u) / scale;
  return __builtin_amdgcn_cvt_pk_fp8_f32(to_range(a), to_range(b), old, kHigh);
}
// A chunk (eight dims) as its pool stores it.
__device__ __forceinline__ void put(u32x4* slot, u32x4 x, float) { *slot = x; }
// One-byte E4M3 pools: every element is divided by its pool's scale in fp32, clamped to the format's range
// (+-448: there is no infinity to overflow to) and rounded to nearest even by the hardware conversion.
__device__ __forceinline__ void put(u32x2* slot, u32x4 x, float scale) {
  u32x2 y;
  y.x = quantise2<true>(x.y, scale, quantise2<false>(x.x, scale, 0));
  y.y = quantise2<true>(x.w, scale, quantise2<false>(x.z, scale, 0));
  *slot = y;
}

template <typename Slot>
__global__ __launch_bounds__(kAppendThreads) void kv_append_kernel(
    AppendTarget a, const u32x4* __restrict__ k_new, const u32x4* __restrict__ v_new, Slot* __restrict__ k_pool,
    Slot* __restrict__ v_pool, float k_scale, float v_scale) {
  const int s = blockIdx.x;
  const int i = blockIdx.y * kAppendThreads + threadIdx.x;
  const bool is_v = i >= a.row_chunks;
  const int e = is_v ? i - a.row_chunks : i;   // chunk of the request's K or V rows: (KV head, chunk of its row)
  const u32x4 x = (is_v ? v_new : k_new)[(int64_t)s * a.row_chunks + min(e, a.row_chunks - 1)];
  typedef const int32_t __attribute__((address_space(4))) * ScalarLoad;   // both look-ups are the same for all lanes
  const int L = min(max(*(ScalarLoad)(a.context_lens + s), 0), a.max_ctx);
  const int t = max(L, 1) - 1;
  // no branch here: an empty request, whose table is not to be read, reads its length again
  const int32_t* entry = a.block_tables + (int64_t)s * a.MAXB + (t >> a.log_block);
  asm volatile("" : : "s"(entry));
  const int id = *(ScalarLoad)(L > 0 ? entry : a.context_lens + s);
  asm volatile("" : : "v"(x), "s"(id), "s"(k_pool), "s"(v_pool));   // asked for before the branches, not in them
  if (L == 0 || e >= a.row_chunks) return;
  if ((unsigned)id >= (unsigned)a.NB) {   // never follow a corrupt id; report it once per request
    if (a.id_faults && i == 0) atomicAdd(a.id_faults, 1);
    return;
  }
  const int64_t row = ((((int64_t)id * a.Hkv + (e >> a.log_chunks)) << a.log_block) + (t & ((1 << a.log_block) - 1)));
  put((is_v ? v_pool : k_pool) + (row << a.log_chunks) + (e & ((1 << a.log_chunks) - 1)), x, is_v ? v_scale : k_scale);
}

template <typename Slot>
hipError_t launch(const uint16_t* k_new, const uint16_t* v_new, void* k_pool, void* v_pool,
                  const int32_t* block_tables, const int32_t* context_lens, float k_scale, float v_scale, int S,
                  int Hkv, int D, int MAXB, int B, int max_ctx, int NB, int32_t* id_faults, hipStream_t stream) {
  const AppendTarget a = {block_tables,          context_lens,      id_faults, Hkv * (D / 8),
                          __builtin_ctz(D / 8), __builtin_ctz(B), MAXB,      Hkv, max_ctx, NB};
  const int chunks = 2 * a.row_chunks;
  const dim3 block(chunks < kAppendThreads ? (chunks + 63) / 64 * 64 : kAppendThreads);
  const dim3 grid(S, (chunks + kAppendThreads - 1) / kAppendThreads);
  hipLaunchKernelGGL(kv_append_kernel<Slot>, grid, block, 0, stream, a, (const u32x4*)k_new, (const u32x4*)v_new,
                     (Slot*)k_pool, (Slot*)v_pool, k_scale, v_scale);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_kv_append_fp8(const uint16_t* k_new, const uint16_t* v_new, void* k_pool,
                                void* v_pool, const int32_t* block_tables,
                                const int32_t* context_lens, float k_scale, float v_scale, int S,
                                int Hkv, int D, int MAXB, int B, int max_ctx, int NB,
                                int32_t* id_faults, hipStream_t stream) {
  return launch<u32x2>(k_new, v_new, k_pool, v_pool, block_tables, context_lens, k_scale, v_scale, S, Hkv, D, MAXB,
                       B, max_ctx, NB, id_faults, stream);
}

hipError_t launch_kv_append(const uint16_t* k_new, const uint16_t* v_new, uint16_t* k_pool,
                            uint16_t* v_pool, const int32_t* block_tables,
                            const int32_t* context_lens, int S, int Hkv, int D, int MAXB, int B,
                            int max_ctx, int NB, int32_t* id_faults, hipStream_t stream) {
  return launch<u32x4>(k_new, v_new, k_pool, v_pool, block_tables, context_lens, 1.f, 1.f, S, Hkv, D, MAXB, B,
                       max_ctx, NB, id_faults, stream);
}

}  // namespace pkv
