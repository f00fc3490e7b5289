// KV-block gather / scatter for gfx950: whole physical blocks move between a
// paged pool and a contiguous staging image (eviction / reload of a preempted
// request, paper Section II-B; whole-cache migration at the phase boundary,
// Section IV-B).  Pure 16-byte loads and stores, no arithmetic: bit-exact.
#include "pkv_kernels.h"

namespace pkv {
namespace {

// Cache policy.  The pool side is always nontemporal: neither the blocks read
// nor the blocks written are touched again soon, and ordinary stores would leave
// dirty lines whose write-back slows the kernel that runs next (an attention
// call measured 17-30 % slower after such a copy).  The staging side depends on
// the image's size.  An image that fits the 256 MB memory-side cache of an
// MI355X is written with write-through stores and read back with ordinary
// loads, so that the scatter (or the copy engine) that follows finds it on
// chip: gather + scatter of 153 MB per pool run 22 % faster that way (6.66
// instead of 5.44 TB/s read+write), with no effect on the next kernel.  The
// gain holds up to an image of about 280 MB, is gone at 310 MB, and beyond that
// a cached image only evicts itself (8 % slower than streaming at 370 MB), so
// larger images are streamed with nontemporal accesses on both sides.
constexpr int kCopyThreads = 256;
constexpr int64_t kCachedStagingBytes = (int64_t)256 << 20;       // staging images up to this size stay on chip

enum Policy { kStream, kPlain, kWriteThrough };

template <int kPolicy>
__device__ __forceinline__ u32x4 ld16(const u32x4* p) {
  if (kPolicy == kStream) return __builtin_nontemporal_load(p);
  return *p;
}
template <int kPolicy>
__device__ __forceinline__ void st16(u32x4* p, u32x4 v) {
  if (kPolicy == kStream) __builtin_nontemporal_store(v, p);
  else if (kPolicy == kWriteThrough)
    // opaque to the compiler, so the wait states a wide store needs before its data
    // registers may be overwritten are spelled out
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
  else *p = v;
}

// The listed blocks, one after the other, are one row of 16-byte chunks, and a lane moves one of them:
// a copy lives on how many of its loads the chip has under way and how evenly they fall on the memory
// channels, and 4 KiB slices dealt round the compute dies do both better than 32 KiB slices (eight
// chunks per lane, all loads before the first store).  On image sizes from 0.25 to 800 MB and blocks from
// 2 to 128 KiB: 128 KiB blocks, 800 MB: move 327 -> 272 us, scatter 320 -> 273; 32 KiB blocks: scatter
// 321 -> 301, gather 280 -> 270, move 617 and 618 at 750 MB; 2 KiB blocks, 150 MB: 82 -> 66; 5 MB of 16 KiB
// blocks: 5.4 -> 4.4 us.
// More than one chunk, one after the other, where that is faster (chunks_per_lane).
//
// kMode 0: staging[i] = pool[ids_a[i]]; 1: pool[ids_a[i]] = staging[i]; 2: dst[ids_b[i]] = src[ids_a[i]].
// kWhole: a block is a whole number of slices, so the ids are the same for the workgroup and the
// base addresses scalar; otherwise each lane looks its chunk's block up.  Byte offsets are 64-bit (a
// pool passes 2 GiB at the long-context sizes).
template <int kMode, bool kCachedStaging, bool kWhole, int kPer>
__global__ __launch_bounds__(kCopyThreads) void kv_block_copy_kernel(
    const u32x4* __restrict__ src, u32x4* __restrict__ dst, const int32_t* __restrict__ ids_a,
    const int32_t* __restrict__ ids_b, uint32_t chunks_per_block, int64_t src_pool_blocks,
    int64_t dst_pool_blocks, int64_t n_blocks, int64_t slices, int32_t* __restrict__ id_faults) {
  constexpr int kLd = (kMode == 1 && kCachedStaging) ? kPlain : kStream;
  constexpr int kSt = (kMode == 0 && kCachedStaging) ? kWriteThrough : kStream;
  for (int64_t slice = blockIdx.x; slice < slices; slice += gridDim.x) {
    int64_t i;         // listed block
    uint32_t chunk;    // within it
    if (kWhole) {
      const uint32_t per = chunks_per_block / (kCopyThreads * kPer);
      i = slices >> 32 ? slice / per : (int64_t)((uint32_t)slice / per);
      chunk = (uint32_t)(slice - i * per) * (kCopyThreads * kPer) + threadIdx.x;
    } else {
      const int64_t c = slice * kCopyThreads + threadIdx.x;
      i = (slices * kCopyThreads) >> 32 ? c / chunks_per_block : (int64_t)((uint32_t)c / chunks_per_block);
      chunk = (uint32_t)(c - i * chunks_per_block);
      if (i >= n_blocks) continue;
    }
    const int64_t from = kMode == 1 ? i : ids_a[i];
    const int64_t to = kMode == 0 ? i : kMode == 1 ? ids_a[i] : ids_b[i];
    if (from < 0 || from >= src_pool_blocks || to < 0 || to >= dst_pool_blocks) {
      // never follow a corrupt id; the skipped block is reported once
      if (id_faults && chunk == 0) atomicAdd(id_faults, 1);
      continue;
    }
    const u32x4* s = src + from * chunks_per_block + chunk;
    u32x4* d = dst + to * chunks_per_block + chunk;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      st16<kSt>(d + u * kCopyThreads, ld16<kLd>(s + u * kCopyThreads));
      asm volatile("" : : : "memory");   // one after the other: loads ahead of the stores made a gather a third slower
    }
  }
}

// Chunks per lane: two, in blocks of which they fill a whole number, for
//   a scatter of 64 MB or more (us for gather + scatter of two pools in 32 KiB blocks, inputs changing from call
//   to call, 1 / 2 / 4 chunks: 64 MB 86.2 / 85.0 / 85.7, 125 MB 169 / 157 / 160, 143 MB 199 / 202 / 206, 205 MB
//   271 / 257 / 260; 10 MB 21.6 with 1, 24.2 with 4)
//   both ways where the blocks are 8 KiB times an odd number and the image has 4 MB or more (1 / 2: 10 MB
//   21.8 / 20.0, 100 MB 136 / 126; 2 MB 9.9 / 10.8)
int chunks_per_lane(int mode, bool cached, int64_t chunks, int64_t image_bytes) {
  if (!cached || chunks % (2 * kCopyThreads) != 0) return 1;
  const bool odd = chunks % (4 * kCopyThreads) != 0;
  return (odd && image_bytes >= ((int64_t)4 << 20)) || (mode == 1 && image_bytes >= ((int64_t)64 << 20)) ? 2 : 1;
}

template <int kMode>
hipError_t launch(const void* src, void* dst, const int32_t* ids_a, const int32_t* ids_b,
                  int64_t src_pool_blocks, int64_t dst_pool_blocks, int64_t n_blocks,
                  int64_t block_bytes, int32_t* id_faults, hipStream_t stream) {
  const int64_t chunks = block_bytes / 16;   // at most 2^26
  const bool cached = kMode != 2 && n_blocks * block_bytes <= kCachedStagingBytes;
  const bool whole = chunks % kCopyThreads == 0;
  const int per = chunks_per_lane(kMode, cached, chunks, n_blocks * block_bytes);
  const int64_t slices = (n_blocks * chunks + kCopyThreads * per - 1) / (kCopyThreads * per);
  // one workgroup per slice (the hardware dispatcher balances them better than a persistent grid
  // did); a list of more than kMaxGroups slices (32 GiB) is walked with a stride, which keeps the
  // launch below 2^32 work-items
  constexpr int64_t kMaxGroups = (int64_t)1 << 23;
  const dim3 grid((unsigned)(slices > kMaxGroups ? kMaxGroups : slices));
  auto kernel = whole ? kv_block_copy_kernel<kMode, false, true, 1> : kv_block_copy_kernel<kMode, false, false, 1>;
  if constexpr (kMode != 2) {
    if (cached)
      kernel = per == 2 ? kv_block_copy_kernel<kMode, true, true, 2>
               : whole  ? kv_block_copy_kernel<kMode, true, true, 1>
                        : kv_block_copy_kernel<kMode, true, false, 1>;
  }
  hipLaunchKernelGGL(kernel, grid, dim3(kCopyThreads), 0, stream, (const u32x4*)src, (u32x4*)dst,
                     ids_a, ids_b, (uint32_t)chunks, src_pool_blocks, dst_pool_blocks, n_blocks, slices,
                     id_faults);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_copy(const void* src, void* dst, int64_t bytes, hipStream_t stream) {
  return hipMemcpyAsync(dst, src, (size_t)bytes, hipMemcpyDeviceToDevice, stream);
}

hipError_t launch_kv_block_copy(const void* src, void* dst, const int32_t* block_ids,
                                int64_t n_blocks, int64_t block_bytes, int64_t num_pool_blocks,
                                bool gather, int32_t* id_faults, hipStream_t stream) {
  return gather ? launch<0>(src, dst, block_ids, nullptr, num_pool_blocks, n_blocks, n_blocks,
                            block_bytes, id_faults, stream)
                : launch<1>(src, dst, block_ids, nullptr, n_blocks, num_pool_blocks, n_blocks,
                            block_bytes, id_faults, stream);
}

hipError_t launch_kv_block_move(const void* src, const int32_t* src_ids, int64_t src_pool_blocks,
                                void* dst, const int32_t* dst_ids, int64_t dst_pool_blocks,
                                int64_t n_blocks, int64_t block_bytes, int32_t* id_faults,
                                hipStream_t stream) {
  return launch<2>(src, dst, src_ids, dst_ids, src_pool_blocks, dst_pool_blocks, n_blocks,
                   block_bytes, id_faults, stream);
}

}  // namespace pkv
