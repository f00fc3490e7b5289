// Paged decode attention, stream pass, for gfx950 (wave64, MFMA).
//
// Decode attends over every running request's whole KV cache and is bound by
// memory bandwidth (paper Section II-A), and the batch mixes short answering
// contexts with long reasoning ones (Section III), so equal work per wavefront
// cannot come from a per-request grid.  Instead the batch's KV blocks form one
// stream (layout in pkv_kernels.h) that is cut into kStreamWaves equal shares:
// every wavefront reads the same number of blocks (+-1), starts streaming at
// once, never idles between requests, and there is no tail of late workgroups.
// A wavefront computes one partial result per run (a stretch of its share inside
// one request, one KV head and one P-token partition) and folds the runs of one
// (request, KV head) together.  What lies wholly inside its share is finished there and
// then: normalised, rounded and staged in LDS for a burst of stores (512 requests of 16
// to 512 tokens: 1.5 MB of records and their reduce pass instead of 16 MB, call 125 ->
// 115 us).  Of what it shares with other wavefronts it leaves one record, and the
// reduce pass (attn_reduce.hip) combines the records of each (request, KV head).
//
// Two ways to that end, by what the segments are like:
//   workgroups' records   the wavefronts of a workgroup fold what they share in LDS first, so at most
//                    two records per workgroup reach memory (64 requests of 1024..8192 tokens on 40/8 heads:
//                    194.2 us -> 191.0 with the reduce pass; one of 8191 19.1 -> 17.6)
//   cut along them   one workgroup per segment, which meets in LDS and finishes it: no records, and no
//                    reduce pass where the bounds say so beforehand (4 requests of 17..300 tokens on 8/2
//                    heads: 14.0 -> 11.3 us and a launch less on the host).  Few and short ones, up to 3
//                    or 6 blocks per wavefront (short_segment).
//
// Per 16-token block, lane = 16*c + n, head_dim D = 128 (64 and 256 below):
//   S^T = K . Q^T   D/32 v_mfma_f32_16x16x32_bf16 (k = 32 dims each).
//         A = K rows: lane (n, c) has the 16 bytes at dims 32*jj + 8*c of
//         token tau(n) = 4*(n%4) + n/4.  K is loaded in whole rows, 1 KiB in a row per
//         load, and turned to that order in LDS.  B = q: lane (n, c) holds the same dims of head n
//         (the GQA group padded to 16 rows).  The result leaves lane (n, c)
//         with head n's scores for tokens 4*i + c.
//   P     = exp2(score - m) in fp32, split into bf16 hi + lo parts so that the
//         weights keep ~16 mantissa bits through the second product.
//   O    += P . V   D/16 v_mfma_f32_16x16x16_bf16 per part.  V is loaded in its
//         natural order (lane (n, c) gets dims 8n..8n+7 of tokens 4*e + c, four
//         fully contiguous 1 KiB loads); the operand for output dims 8*n + i
//         pairs up the i-th halves of those four loads with v_perm_b32.  The
//         token order 4*e + c is exactly the one the scores came out in, so P
//         needs no shuffle between the two products.
//   D = 64:  lane (n, c) owns dims 4n..4n+3; its V loads are 8 bytes wide (four
//         fully contiguous 512-byte loads), two K steps, four output tiles.
//   D = 256: lane (n, c) owns dims 8n..8n+7 of each 128-dim half; eight K steps,
//         eight 16-byte V loads (a 256-byte run per token per load), sixteen
//         output tiles; a block is 16 KiB here and a wavefront needs more than half
//         of a SIMD's registers, so one wavefront per SIMD streams (half as many).
// The running maximum m is only raised when a score exceeds it by more than
// 2^kLazyLog2; any reference value gives the same softmax, and the bound keeps
// every weight within fp32/bf16 range.
//
// Where a block lives (physical id, KV head), how many of its tokens are valid
// and whether it closes a run is worked out 64 blocks at a time, one block per
// lane ("descriptors"), one window ahead of use; the streaming loop itself only
// reads a lane of those registers per block, so no memory access sits on the
// address path of the KV loads.
//
// Memory traffic.  The KV loads of a block (eight of 16 bytes at D = 128) are
// nontemporal and unconditional.  A load that takes 64 bytes of each of 16 tokens, as the matrix cores
// want K, keeps the address unit busy for twice the lines and takes each of them from the caches in two
// halves; whole rows and a turn in LDS (no bank conflicts, 32 KiB a workgroup) cost a few hundred cycles of
// latency per block.  With the order of the loads below, append and attention, us before / after: 4 requests of 17..300
// tokens 12.2 / 11.5, one of 8191 18.2 / 17.1, 8 at D = 256 35.0 / 33.5, 32 at D = 64 44.1 / 41.8, 64 on 8-bit pools 105.0 /
// 103.9; where the memory is saturated 64 of 1024..8192 189.1 / 188.8, 128 long ones 592.4 / 588.8.  In operand order all the
// same: D = 128 without room in LDS (stream_lds), e4m3 at D = 64, and large batches in e4m3 at D = 256 (large_at_256).
// What is in flight per wavefront, 2048 of them (1024 at D = 256):
//   e4m3 at D = 64 (blocks of 2 KiB): the next block's loads go out before this one's are waited for (once they are there
//       instead: 20 requests of 12000..16500 tokens on 40/8 heads 63.8 us, this way 61.3; 20 of 21000..28000 98.6 and 95.3)
//   bf16 at D = 64 and e4m3 at D = 128 (4 KiB), e4m3 at D = 256 (8 KiB), bf16 there in small batches (16 KiB): the next block's
//       loads go out once this one's are there
//   bf16 at D = 128 (8 KiB) and in large batches at D = 256 (kLate): V of this block and kAhead loads of the next one's K go
//       out once K is there, the rest of that K after the block, at D = 128 4 to 6 KiB at any time, 8 in short shares.  With 8 KiB some dies of the
//       chip get more than their part and the others end late (64 requests 191.9 us instead of 188.9, 128 long ones 584
//       instead of 578; with 4 KiB 4-KiB blocks lose a quarter, which is why those have all of theirs ahead)
// Deeper rings (3 or 7 blocks ahead) only lengthen the queues.
// Finished rows and records wait in LDS and are written in
// bursts of full-width write-through stores that the compiler's wait-count
// bookkeeping does not see (see store16).
#pragma once

#include "attn_partial.h"
#include "pkv_kernels.h"

#include <type_traits>

namespace pkv {
namespace {

constexpr int kWindow = 64;       // descriptors per window: one per lane

// What depends on the head dimension and the pool format.
template <int kD, bool kFp8> struct Dim;
template <> struct Dim<64, false> {
  static constexpr int kKSteps = 2, kKLoads = 2, kVLoads = 4, kTiles = 4, kElemBytes = 2;
  typedef uint32_t VReg __attribute__((ext_vector_type(2)));
};
template <> struct Dim<128, false> {
  static constexpr int kKSteps = 4, kKLoads = 4, kVLoads = 4, kTiles = 8, kElemBytes = 2;
  typedef uint32_t VReg __attribute__((ext_vector_type(4)));
};
template <> struct Dim<256, false> {
  static constexpr int kKSteps = 8, kKLoads = 8, kVLoads = 8, kTiles = 16, kElemBytes = 2;
  typedef uint32_t VReg __attribute__((ext_vector_type(4)));
};
// K and V stored as one-byte e4m3 values: the values are widened to bf16 (exactly) in
// registers and then take the same path as a bf16 pool.  A K load is 16 bytes = 16 dims of one token and feeds two MFMA steps; a V load is
// the lane's dims of one token (4 bytes at D = 64, 8 bytes otherwise).
template <> struct Dim<64, true> {
  static constexpr int kKSteps = 2, kKLoads = 1, kVLoads = 4, kTiles = 4, kElemBytes = 1;
  typedef uint32_t VReg;
};
template <> struct Dim<128, true> {
  static constexpr int kKSteps = 4, kKLoads = 2, kVLoads = 4, kTiles = 8, kElemBytes = 1;
  typedef uint32_t VReg __attribute__((ext_vector_type(2)));
};
template <> struct Dim<256, true> {
  static constexpr int kKSteps = 8, kKLoads = 4, kVLoads = 8, kTiles = 16, kElemBytes = 1;
  typedef uint32_t VReg __attribute__((ext_vector_type(2)));
};
// First dim of output tiles 4t..4t+3 (they are consecutive dims) in the lane of column n.
template <int kD> __device__ __forceinline__ int tile_group_dim(int t, int n) {
  if (kD == 64) return 4 * n;
  if (kD == 128) return 8 * n + 4 * t;
  return 128 * (t >> 1) + 8 * n + 4 * (t & 1);
}
constexpr float kLazyLog2 = 8.f;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

// The same rounding, then the fp32 value of what was kept.
__device__ __forceinline__ float bf16_round(float x, uint32_t& bits) {
  bits = pack_bf16(x, 0.f) & 0xffffu;
  return __uint_as_float(bits << 16);
}

// Four e4m3 bytes of one dword -> four bf16 (exact: every e4m3 value is a bf16 value), an instruction for two of them.  By way of
// fp32 it took two: 72 shapes at D = 64 0.983 of the time, 18 of 8 to 70 blocks a wavefront at D = 128 0.996, 64 requests of
// 1024..8192 tokens 102.2 -> 101.5 us.
__device__ __forceinline__ u32x2 widen_e4m3x4(uint32_t w) {
  return u32x2{__builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)w, 1.f, false)),
               __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)w, 1.f, true))};
}

// Stores of finished rows and of records.  They are written as opaque instructions on
// purpose: gfx9-family hardware counts loads and stores in one counter, and once
// the compiler knows a store is pending it can no longer wait for "all but the N
// youngest loads" and drains the whole ring of KV loads at the next use.  Hidden
// from that bookkeeping, a wait sized for the loads alone is still sufficient
// (loads retire in order among themselves, so extra pending stores only make the
// same wait stricter), and the record itself is only read by the next kernel.
// sc1 makes the store write through instead of leaving a dirty line behind for a
// later eviction (measured while records were still written once per partition:
// 512-token partitions then cost 8 % instead of 13 % on the long-context batch).
__device__ __forceinline__ void store16(void* p, u32x4 v) {
  // the trailing s_nop covers the wait states a wide store needs before a vector
  // op may overwrite its data registers (the compiler cannot see that this is a store)
  asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
}

// A nontemporal load of a buffer, zero out of its bounds.
constexpr int kRawBuffer = 0x00020000;   // last word of the buffer's descriptor: bytes
template <typename T>
__device__ __forceinline__ T load_nt(__amdgpu_buffer_rsrc_t b, int offset) {
  constexpr int kNt = 2;
  if constexpr (sizeof(T) == 16) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b128(b, offset, 0, kNt));
  else if constexpr (sizeof(T) == 8) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(b, offset, 0, kNt));
  else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(b, offset, 0, kNt));
}

// One window of block descriptors: lane i describes stream index jbase + i.
struct Window {
  int slab;   // which slab (16 tokens of one KV head; 4 KiB at D = 128 in bf16), counted from the pool's start; 0 when not read
  int meta;   // bits 0-7 valid tokens (0..16), then the kMeta flags
  int seg;    // s * Hkv + kvh: the segment, whose first query/output row is seg * G
};
// A position of the stream: block b of the nb blocks of request s, KV head kvh.
struct Place {
  int s, kvh, b, nb;
};

constexpr int kMetaLast = 1 << 8;       // closes a run
constexpr int kMetaSegFirst = 1 << 9;   // first block of its segment in this share
constexpr int kMetaSegEnd = 1 << 10;    // last block of its segment
constexpr int kMetaOpenLeft = 1 << 11;  // its segment begins before this share

// How a wavefront's share ends.
constexpr int kEndsLeft = 1;      // the left record is in use: the first segment begins before the share
constexpr int kEndsThrough = 2;   // and goes on after it
constexpr int kEndsRight = 4;     // the right record is in use: the last segment begins in the share and goes on

// Inclusive prefix sum over the wavefront, in the vector unit.  It stands before the first load of the stream: by six shuffles
// through LDS, 4 requests of 17..300 tokens took 11.5 us for append and attention, this way 11.3; one of 8191 17.2 and 16.95.
__device__ __forceinline__ int wave_prefix(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);    // row_shr:1, 2, 4, 8 within 16 lanes
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // lane 15 of each row to the next row: rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // lane 31 to rows 2 and 3
  return x;
}

// The launch descriptor once more, from the kernel's argument block: what only the merge needs
// is then loaded after the stream and does not take up scalar registers during it.
__device__ __forceinline__ const AttnLaunch& reread(const AttnLaunch&) {
  typedef const AttnLaunch __attribute__((address_space(4))) * ArgPtr;
  ArgPtr p = (ArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const AttnLaunch*)p;
}

// WholeLayer: the bounds say that each segment has a workgroup.  Where its blocks are then follows from its request's length alone, which
// is asked for together with the query group: no prefix sums, no search, no barrier before the first K.  Append and attention against the
// general kernel, which finds out on the device: 4 requests of 17..300 tokens on 8/2 heads 10.8 -> 8.75 us, geometric means of 100 shapes
// each (1 to 250 segments of 10 to 300 tokens) D = 64 0.79, e4m3 there 0.79, D = 128 0.80 and 0.81, D = 256 0.85 and 0.85, measured with the
// table row asked for together with the length as well.  That took 0.1 to 0.3 us less, but reads entries behind a request's last block,
// which the caller is promised are not read.
// kLarge: as large batches want it (large_at_256; at D = 128 in bf16 all but short ones, short_at_128).
template <int kD, bool kFp8, typename Layers, bool kLarge>
__global__ __launch_bounds__(group_waves(kD) * 64) void attn_stream_kernel(AttnLaunch a, Layers layers) {
  typedef Dim<kD, kFp8> DD;
  typedef typename DD::VReg VReg;                 // one V load as it arrives
  typedef typename Dim<kD, false>::VReg VOp;      // the same rows as bf16
  constexpr int kKSteps = DD::kKSteps, kKLoads = DD::kKLoads, kVLoads = DD::kVLoads,
                kTiles = DD::kTiles, kElemBytes = DD::kElemBytes;
  // V goes out when K is there, not a block ahead, and with it some of the next block's K loads: kAhead, or all where shares are
  // short (short_at_128; AttnLayers have a workgroup for each short segment).
  constexpr bool kLate = !kFp8 && (kD == 128 || (kD == 256 && kLarge));
  constexpr bool kWhole = std::is_same_v<Layers, WholeLayer>;
  constexpr int kNextK = kD == 128 && (!kLarge || std::is_same_v<Layers, AttnLayers>) ? kKLoads : kAhead;
  constexpr bool kTwoBlocks = kD == 64 && kFp8;   // the next block's loads go out before this one's have arrived
  constexpr int kGroupWaves = group_waves(kD), kThreads = kGroupWaves * 64;
  extern __shared__ __align__(16) int smem[];
  int* cumB = smem;                  // [S+1] blocks before request s
  int* lens = smem + (a.S + 1);      // [S]   clamped context lengths
  // then, 16-byte aligned, each wavefront's left record and its right record; the right
  // record shares its room with finished rows that wait to be stored
  const int rec_floats = record_floats(a.G, kD);
  float* wave_lds = (float*)(smem + ((2 * (a.S + 1) + 3) & ~3));
  __shared__ int share_ends[kGroupWaves];   // how each wavefront's share ends
  __shared__ SharedSegment word;          // the workgroup's, for the reduce pass
  __shared__ int left_seg[kGroupWaves];   // the segment that the share's first block belongs to
  __shared__ int any_long;                // with more than 64 requests
  __shared__ int sum64[kMaxSeqs / 64];   // blocks of each 64 requests

  constexpr bool kChained = std::is_same_v<Layers, ChainedLayers>;   // a workgroup streams its range of one layer after the other
  int of = layer_index(layers);   // layer
  AttnLayer layer = layer_of(a, layers);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int n = lane & 15, c = lane >> 4;
  const int G = a.G, S = a.S, Hkv = a.Hkv;
  const int bpp = a.P / kBlockTokens;   // blocks per partition
  float* rec_left = wave_lds + wave * a.wave_lds_floats;
  float* rec_right = rec_left + rec_floats;
  uint16_t* staged = (uint16_t*)rec_right;

  int T = 0, W = 0, first_wave = 0, last_wave = -1, pos0 = 0, nshare = 0;
  int own_len = 0, own_start = 0;   // up to 64 requests: lane s's context length and first position
  bool whole = kWhole;
  const int groups = a.waves / kGroupWaves;   // of the layer
  const int w = blockIdx.x * kGroupWaves + wave;
  u32x4 qnext[kKSteps];
  int seg = 0, seg_next = 0;   // the segment being streamed, and the one of the query group that was asked for last
  auto load_q = [&](int segment) {
    seg_next = segment;
    const u32x4* qrow_p = (const u32x4*)(layer.q + (int64_t)(segment * G + min(n, G - 1)) * kD);
#pragma unroll
    for (int jj = 0; jj < kKSteps; ++jj)
      // dims of step jj in this lane: 32*jj + 8*c .. +7, or, following the byte order of an
      // e4m3 K load, 64*(jj/2) + 16*c + 8*(jj%2) .. +7
      qnext[jj] = kFp8 ? qrow_p[8 * (jj >> 1) + 2 * c + (jj & 1)] : qrow_p[4 * jj + c];
  };
  if constexpr (!kWhole) {
    // Prefix sums over the requests.  Up to 64: every wavefront for itself, all to the same place and the same values, so that none
    // waits for another.  More: 64 to a wavefront at a time, first within each 64, then the sums of the 64s before them (512
    // requests in turns of one wavefront took 3.6 us to get here; with the empty window below left out, the call 114.1 -> 111.7 us).
    int longest = 0, blocks = 0;
    // What else the start needs of the launch descriptor is asked for with the lengths; where it is used it would be waited for,
    // one word after the other.  With no request's data read back from LDS up to 64 requests: one of 8191 tokens 16.7 -> 16.5 us, 64 of
    // 64 on 40/8 heads 11.6 -> 11.45, 64 of 1024..8192 on 8-bit pools 101.7 -> 101.0; 696 shapes of up to 4 blocks a share 0.986.
    asm volatile("" : : "s"(a.waves), "s"(a.short_blocks), "s"(a.max_ctx), "s"(a.context_lens), "s"(a.block_tables), "s"(a.MAXB),
                 "s"(a.NB), "s"(a.upb), "s"(a.P), "s"(layer.q), "s"(layer.k_pool), "s"(layer.v_pool), "s"(a.wave_lds_floats));
    for (int base = S > 64 ? 64 * wave : 0; base < S; base += kThreads) {
      const int i = base + lane;
      const int L = (i < S) ? min(max(a.context_lens[i], 0), a.max_ctx) : 0;
      const int nb = (L + kBlockTokens - 1) / kBlockTokens;
      longest = max(longest, nb);
      const int xb = wave_prefix(nb);
      if (i < S) { lens[i] = L; cumB[i] = xb - nb; }
      if (lane == 63) { if (S <= 64) cumB[S] = xb; else sum64[base >> 6] = xb; }
      blocks = xb;
      own_len = L;
      own_start = i < S ? Hkv * (xb - nb) : INT32_MAX;
    }
    __builtin_amdgcn_wave_barrier();
    bool some_long = __any(longest > a.short_blocks);
    blocks = __builtin_amdgcn_readlane(blocks, 63);
    if (S > 64) {
      if (threadIdx.x == 0) any_long = 0;
      __syncthreads();
      if (some_long && lane == 0) any_long = 1;
      // lane c: all requests before the c-th 64 (kMaxSeqs = 32 of them)
      const int mine = lane < (S + 63) >> 6 ? sum64[lane] : 0;
      int before = wave_prefix(mine);
      if (threadIdx.x == 63) cumB[S] = before;
      blocks = __builtin_amdgcn_readlane(before, 63);
      before -= mine;
      for (int base = 64 * wave; base < S; base += kThreads) {
        const int add = __shfl(before, base >> 6);
        if (base > 0 && base + lane < S) cumB[base + lane] += add;
      }
      __syncthreads();
      some_long = __builtin_amdgcn_readfirstlane(any_long);
    }

    // Equal shares: every participating wavefront gets at least one block, so that consecutive
    // runs of a segment always belong to the same or to adjacent wavefronts.  A batch of a few
    // short segments is cut along the segments instead, one to a workgroup (see short_segment).
    T = Hkv * blocks;
    whole = !some_long && S * Hkv <= groups;
    if (__builtin_expect(whole, 0)) {
      const int s = (int)blockIdx.x / Hkv, kvh = (int)blockIdx.x - s * Hkv;
      const int nb = s < S ? cumB[s + 1] - cumB[s] : 0;
      W = min(kGroupWaves, nb);
      first_wave = 0;
      last_wave = W - 1;
      if (wave < W) {
        const ShareMap shares(nb, W);
        pos0 = Hkv * cumB[s] + kvh * nb + shares.start(wave);
        nshare = shares.start(wave + 1) - shares.start(wave);
      }
    } else {
      W = share_count(T, a.waves);
      first_wave = blockIdx.x * kGroupWaves;
      last_wave = min(kGroupWaves, W - first_wave) - 1;
      if (w < W) {
        const ShareMap shares(T, W);
        pos0 = shares.start(w);
        nshare = shares.start(w + 1) - pos0;
      }
    }
  }
  // What lies where each segment has a workgroup.
  int whole_len = 0, whole_entry = 0;
  if constexpr (kWhole) {
    const int s = blockIdx.z;
    load_q(s * Hkv + blockIdx.x);
    typedef const int32_t __attribute__((address_space(4))) * ScalarLoad;
    whole_len = min(max(*(ScalarLoad)(a.context_lens + s), 0), a.max_ctx);
    const int nb = (whole_len + kBlockTokens - 1) / kBlockTokens;
    if (nb == 0) {   // an empty request owes zero rows
      uint32_t* dst = (uint32_t*)(layer.out + (int64_t)seg_next * G * kD);
      for (int f = threadIdx.x; f < G * kD / 2; f += kThreads) dst[f] = 0;
      return;
    }
    if (lane * a.upb < nb) whole_entry = a.block_tables[(int64_t)s * a.MAXB + lane];   // entries behind the last block are never read
    W = min(kGroupWaves, nb);
    last_wave = W - 1;
    if (wave < W) {
      const ShareMap shares(nb, W);
      pos0 = shares.start(wave);
      nshare = shares.start(wave + 1) - pos0;
    }
  }
  // the same for all lanes: the stream's loop and its addresses are scalar (32 requests at D = 64 43.6 -> 43.1 us)
  pos0 = __builtin_amdgcn_readfirstlane(pos0);
  nshare = __builtin_amdgcn_readfirstlane(nshare);
  // An empty request owes zero rows.
  auto zero_empty_rows = [&]() {
    for (int s = w; s < S; s += groups * kGroupWaves) {
      if (cumB[s + 1] != cumB[s]) continue;
      uint32_t* dst = (uint32_t*)(layer.out + (int64_t)s * a.Hq * kD);
      for (int f = lane; f < a.Hq * kD / 2; f += 64) dst[f] = 0;
    }
  };

  // Is there a reduce pass?  AttnLayers have a workgroup for each segment, too.
  constexpr bool kLeavesWords = !kWhole && !std::is_same_v<Layers, AttnLayers>;
  if (!kWhole && __builtin_expect(last_wave < 0, 0)) {   // nothing for this workgroup
    for (;;) {
      if (threadIdx.x == 0 && kLeavesWords) shared_segment(a, of, blockIdx.x)->told = 0;
      zero_empty_rows();
      if (!kChained || ++of == layer_count(layers)) return;
      layer = layer_at(a, layers, of);
    }
  }

  int refused = 0;   // table entries outside the pool met while describing this share
  // The request of a position that is the same for all lanes, the largest s with Hkv * cumB[s] <= pos: all in one look, or two
  // with more than 64 of them.
  auto request_of = [&](int pos) -> int {
    if (S <= 64) return __popcll(__ballot(own_start <= pos)) - 1;
    const int start64 = Hkv * cumB[min(64 * lane, S)];
    const int base = 64 * __popcll(__ballot((64 * lane < S) & (start64 <= pos))) - 64;
    const int start = Hkv * cumB[min(base + lane, S)];
    return base + __popcll(__ballot((base + lane < S) & (start <= pos))) - 1;
  };
  struct Request {
    int start, nb, len;   // first position, blocks, tokens
  };
  auto request = [&](int s) -> Request {   // each lane's
    return Request{Hkv * cumB[s], cumB[s + 1] - cumB[s], lens[s]};
  };
  auto the_request = [&](int s) -> Request {   // the same for all lanes
    if (S > 64) return request(s);
    const int len = __builtin_amdgcn_readlane(own_len, s);
    return Request{__builtin_amdgcn_readlane(own_start, s), (len + kBlockTokens - 1) / kBlockTokens, len};
  };
  auto place = [&](int pos, int s, const Request& r) -> Place {
    // o / nb, which is less than Hkv (at most kMaxHeads): the estimate is off by less than one
    const int o = pos - r.start;
    int kvh = (int)((float)o * __builtin_amdgcn_rcpf((float)r.nb)), b = o - kvh * r.nb;
    const bool less = b < 0;
    kvh -= less;
    b += less ? r.nb : 0;
    const bool more = b >= r.nb;
    return Place{s, kvh + more, more ? b - r.nb : b, r.nb};
  };
  const int upb_bits = 31 - __clz(a.upb);
  // Descriptors of stream indices jb .. jb+63 of this share.
  auto describe = [&](int jb) __attribute__((always_inline)) -> Window {
    const int j = jb + lane;
    const bool live = j < nshare;
    const int pos = pos0 + max(min(j, nshare - 1), 0);
    // the requests that the window reaches over, one as a rule, then each lane's among them
    int s = request_of(pos0 + jb);
    const int s_last = request_of(pos0 + max(min(jb + kWindow, nshare) - 1, 0));
    Request r;
    if (s == s_last) {
      r = the_request(s);
    } else {
      for (int step = 1 << (31 - __clz(s_last - s)); step > 0; step >>= 1) {
        const int t = min(s + step, s_last);
        if (Hkv * cumB[t] <= pos) s = t;
      }
      r = request(s);
    }
    const Place at = place(pos, s, r);
    const int kvh = at.kvh, b = at.b, nb = at.nb;
    int ntok = min(kBlockTokens, r.len - kBlockTokens * b);
    // unit b of the request lies in physical block b / upb, at unit b % upb of the KV head's rows
    const int tb = b >> upb_bits;
    const int id = live ? a.block_tables[(int64_t)s * a.MAXB + tb] : -1;
    const bool mapped = (unsigned)id < (unsigned)a.NB;   // ids outside the pool are never followed
    if (!mapped) ntok = 0;
    refused += __popcll(__ballot(live && !mapped));
    Window d;
    d.slab = mapped ? ((id * Hkv + kvh) << upb_bits) + (b - (tb << upb_bits)) : 0;
    bool last = (b + 1 == nb) || (j + 1 == nshare);
    if (__any(nb > bpp)) last |= (unsigned)(b + 1) % (unsigned)bpp == 0;
    const bool seg_first = (b == 0) || (j == 0);
    d.meta = ntok | (last ? kMetaLast : 0) | (seg_first ? kMetaSegFirst : 0) |
             (b + 1 == nb ? kMetaSegEnd : 0) | (b > j ? kMetaOpenLeft : 0);
    if (!live) d.meta = 0;
    d.seg = s * Hkv + kvh;
    return d;
  };

  // The blocks of a wavefront that has its part of one segment: all in one window, their table entries in the lanes' hands.
  auto describe_whole = [&]() -> Window {
    const bool live = lane < nshare;
    const int b = pos0 + lane, tb = b >> upb_bits;
    const int id = __shfl(whole_entry, tb);   // by all lanes: the entries are in lanes that may have no block
    const bool mapped = live && (unsigned)id < (unsigned)a.NB;
    refused += __popcll(__ballot(live && !mapped));
    Window d;
    d.slab = mapped ? (((id * Hkv + (int)blockIdx.x) << upb_bits) + (b - (tb << upb_bits))) : 0;
    const bool ends = 16 * (b + 1) >= whole_len;
    const bool last = ends || ((b + 1) % bpp == 0) || (lane + 1 == nshare);
    d.meta = !live ? 0
                   : (mapped ? min(kBlockTokens, whole_len - kBlockTokens * b) : 0) | (last ? kMetaLast : 0) |
                         (lane == 0 ? kMetaSegFirst : 0) | (ends ? kMetaSegEnd : 0) | (pos0 > 0 ? kMetaOpenLeft : 0);
    d.seg = seg_next;
    return d;
  };
  Window dA;
  if constexpr (kWhole) dA = describe_whole();
  else dA = describe(0);
  Window dB = {0, 0, 0};   // described when the first blocks have been consumed (below)
  int jbase = 0;           // stream index of window A's first block

  const int64_t slab_bytes = (int64_t)kBlockTokens * kD * kElemBytes;  // one (block, KV head) slab
  const int tau = turn_token(n);
  // K, in 16-byte pieces of the slab: a wavefront's load is 64 of them in a row, turned in LDS (turn_place).  Straight in
  // operand order, 4 of each token, where that is all of a token's (e4m3 at D = 64), where LDS has no room (stream_lds), and in
  // large batches in e4m3 at D = 256.
  constexpr int kPieces = kD * kElemBytes / 16;   // of a token
  const bool turns = kD == 128 ? a.turns : !kFp8 || (kD == 256 && !kLarge);
  const int koff = turns ? lane : tau * kPieces + c;
  u32x4* turn = (u32x4*)(wave_lds + kGroupWaves * a.wave_lds_floats) + wave * (kBlockTokens * kPieces);
  // V, in units of one VReg: token 4*e + c, this lane's dims (of half h when D = 256)
  const int voff = kD == 256 ? 32 * c + n : lane;

  u32x4 qop[kKSteps];  // q as the B operand: dims 32*jj + 8*c .. +7 of head n; zero rows beyond the group
  float m = kNegInf;   // running reference maximum of head n (log2 units), same in all four c groups
  float l = 0.f;       // this lane's share of the softmax denominator
  f32x4 o[kTiles];     // o[i][r]: head 4*c + r, dim tile_group_dim(i / 4, n) + i % 4
#pragma unroll
  for (int i = 0; i < kTiles; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};

  // The streaming loop reads a block's descriptor once, when its first loads go out, and keeps it until the block has been consumed.
  struct Block {
    int slab, meta;   // of a Window
  };
  auto block_at = [&](int j) {
    return Block{__builtin_amdgcn_readlane(dA.slab, j - jbase), __builtin_amdgcn_readlane(dA.meta, j - jbase)};
  };
  // The loads of a block, nontemporal: the stream is read once and must not allocate in the
  // caches it passes through.  The loads are unconditional so that every wait in the loop knows
  // exactly how many are outstanding, and their bounds are the block's valid rows: what lies behind a
  // request's last token, a block that is unmapped and an index past the share's end are not read and arrive as zeros.
  // Against whole blocks, the first one of the pool past a share's end, and descriptors looked up for each load: 512 requests of
  // 16..512 tokens 109.5 -> 106.0 us, shares of 1 to 4 blocks at D = 128 0.98 of the time, 72 shapes of 8-bit pools at D = 64 0.983.
  auto rows_of = [&](const void* pool, Block at) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)pool + at.slab * slab_bytes), 0,
                                             (at.meta & 0xff) * (kD * kElemBytes), kRawBuffer);
  };
  auto issue_k = [&](u32x4 (&k)[kKLoads], Block at, int from, int to) {
    const __amdgpu_buffer_rsrc_t b = rows_of(layer.k_pool, at);
    if (turns) {
#pragma unroll
      for (int jj = from; jj < to; ++jj) k[jj] = load_nt<u32x4>(b, 16 * (koff + 64 * jj));
    } else {
#pragma unroll
      for (int jj = from; jj < to; ++jj) k[jj] = load_nt<u32x4>(b, 16 * (koff + 4 * jj));
    }
  };
  auto issue_v = [&](VReg (&v)[kVLoads], Block at) {
    const __amdgpu_buffer_rsrc_t b = rows_of(layer.v_pool, at);
    constexpr int kBytes = sizeof(VReg);
    if (kD == 256) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[2 * e] = load_nt<VReg>(b, kBytes * (voff + 128 * e));
        v[2 * e + 1] = load_nt<VReg>(b, kBytes * (voff + 128 * e + 16));
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = load_nt<VReg>(b, kBytes * (voff + 64 * e));
    }
  };
  // K of a block that has arrived, into LDS and back as the A operand: load L of lane (n, c) is piece 4L + c of token tau(n).
  auto turn_k = [&](u32x4 (&k)[kKLoads]) {
    if (turns) {
#pragma unroll
      for (int jj = 0; jj < kKLoads; ++jj) {
        const int at = 64 * jj + lane;
        turn[turn_place(kPieces, at / kPieces, at % kPieces)] = k[jj];
      }
#pragma unroll
      for (int jj = 0; jj < kKLoads; ++jj) k[jj] = turn[turn_place(kPieces, tau, 4 * jj + c)];
    }
  };

  // Finished rows wait in LDS and go out several segments at a time, and the rest when
  // the share is done.  A store in the middle of the stream is expensive out of
  // proportion to its size: loads and stores retire through one counter, so the KV loads
  // issued after it cannot be consumed before it has been acknowledged, and that costs one
  // stall of several microseconds per burst of stores however few bytes it carries.
  int nstaged = 0;       // finished segments whose rows are in LDS
  int staged_segs = 0;   // lane r: staged segment r
  bool seg_open = false;   // a parked record belongs to the segment being streamed
  int ends_flags = 0, left = 0, right = 0;   // how the share ends, and the segments in the left and the right record
  auto store_staged = [&]() __attribute__((always_inline)) {
    for (int r = 0; r < nstaged; ++r) {
      const int seg = __builtin_amdgcn_readlane(staged_segs, r);
      float* dst = (float*)(layer.out + (int64_t)seg * (G * kD));
      const float* src = (const float*)(staged + r * G * kD);
      for (int f = 4 * lane; f < G * kD / 2; f += 256) store16(dst + f, *(const u32x4*)(src + f));
    }
    nstaged = 0;
  };

  auto consume = [&](u32x4 (&kraw)[kKLoads], VReg (&vraw)[kVLoads], int meta) __attribute__((always_inline)) {
    // The MFMA operands.  bf16 pools: the registers as they are.  e4m3 pools: piece 4L + c of
    // K's row holds dims 16*(4L + c) .. +15 of token tau(n), which feed steps 2L and 2L + 1 (the
    // contraction order is free as long as q follows it, see below); a V load holds the same
    // token and dims as in a bf16 pool, one byte each.
    u32x4 k[kKSteps];
    VOp v[kVLoads];
#pragma unroll
    for (int jj = 0; jj < kKLoads; ++jj) {
      const u32x4 x = kraw[jj];
      if constexpr (kFp8) {
        const u32x2 y[4] = {widen_e4m3x4(x.x), widen_e4m3x4(x.y), widen_e4m3x4(x.z), widen_e4m3x4(x.w)};
        k[2 * jj] = u32x4{y[0].x, y[0].y, y[1].x, y[1].y};
        k[2 * jj + 1] = u32x4{y[2].x, y[2].y, y[3].x, y[3].y};
      } else {
        k[jj] = x;
      }
    }
#pragma unroll
    for (int e = 0; e < kVLoads; ++e) {
      if constexpr (!kFp8) {
        v[e] = vraw[e];
      } else if constexpr (kD == 64) {
        v[e] = widen_e4m3x4(vraw[e]);
      } else {
        const u32x2 a2 = widen_e4m3x4(vraw[e].x), b2 = widen_e4m3x4(vraw[e].y);
        v[e] = VOp{a2.x, a2.y, b2.x, b2.y};
      }
    }
    const int ntok = meta & 0xff;

    f32x4 sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int jj = 0; jj < kKSteps; ++jj)
      sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k[jj]),
                                                   __builtin_bit_cast(bf16x8, qop[jj]), sc, 0, 0, 0);
    float x[4] = {sc.x * a.scale_log2e, sc.y * a.scale_log2e, sc.z * a.scale_log2e,
                  sc.w * a.scale_log2e};
    const bool edge = ntok < kBlockTokens;
    bool valid[4] = {true, true, true, true};
    if (edge) {
      // Last block of a request, or an unmapped one: the rows behind it are zeros, and their
      // scores and weights are replaced by select.  Element e of this lane is token 4*e + c.
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        valid[e] = 4 * e + c < ntok;
        x[e] = valid[e] ? x[e] : kNegInf;
      }
    }
    const float mx = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
    if (__any(mx > m + kLazyLog2)) {
      float mg = fmaxf(mx, __shfl_xor(mx, 16));
      mg = fmaxf(mg, __shfl_xor(mg, 32));
      const float mnew = fmaxf(m, mg);   // finite: some lane of the head saw a valid token
      const float alpha = __builtin_amdgcn_exp2f(m - mnew);
      l *= alpha;
      float ar[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) ar[r] = __shfl(alpha, 4 * c + r);
#pragma unroll
      for (int i = 0; i < kTiles; ++i) {
        o[i].x *= ar[0]; o[i].y *= ar[1]; o[i].z *= ar[2]; o[i].w *= ar[3];
      }
      m = mnew;
    }
    float pw[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) pw[e] = __builtin_amdgcn_exp2f(x[e] - m);
    if (edge) {
#pragma unroll
      for (int e = 0; e < 4; ++e) pw[e] = valid[e] ? pw[e] : 0.f;   // m may still be -inf here
    }
    l += (pw[0] + pw[1]) + (pw[2] + pw[3]);

    // P = hi + lo in bf16.
    uint32_t hb[4];
    float lo[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) lo[e] = pw[e] - bf16_round(pw[e], hb[e]);
    const u32x2 phi = {hb[0] | (hb[1] << 16), hb[2] | (hb[3] << 16)};
    const u32x2 plo = {pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3])};
    const s16x4 pa = __builtin_bit_cast(s16x4, phi);
    const s16x4 pb = __builtin_bit_cast(s16x4, plo);
#pragma unroll
    for (int i = 0; i < kTiles; ++i) {
      // tile i needs, for tokens 4*e + c (e = 0..3), the bf16 of its dim: half (i & 1) of
      // word ((i % 8) >> 1) of the load that holds token e (and, for D = 256, half i / 8)
      const int wsel = (i & 7) >> 1, h = kD == 256 ? i >> 3 : 0, st = kD == 256 ? 2 : 1;
      const uint32_t sel = (i & 1) ? 0x07060302u : 0x05040100u;
      const u32x2 vb = {__builtin_amdgcn_perm(v[st + h][wsel], v[h][wsel], sel),
                        __builtin_amdgcn_perm(v[3 * st + h][wsel], v[2 * st + h][wsel], sel)};
      const s16x4 vop = __builtin_bit_cast(s16x4, vb);
      o[i] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pa, vop, o[i], 0, 0, 0);
      o[i] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pb, vop, o[i], 0, 0, 0);
    }

    if (meta & kMetaLast) {
      // The run ends here.  A segment that lies wholly inside the share is finished now:
      // its rows are normalised, rounded and staged.  Of a segment that other wavefronts
      // share, or of which more partitions follow, the partial result is parked in a
      // record in LDS (the left one when the segment begins before the share, else the
      // right one); a later run of the same segment (the next P-token partition) is folded
      // into it with the split-K merge formula, so there is one record per (wavefront,
      // segment) however small P is.
      const bool open_left = meta & kMetaOpenLeft;
      const bool done = (meta & kMetaSegEnd) && !open_left;
      float* rec = open_left ? rec_left : rec_right;
      float lt = l + __shfl_xor(l, 16);
      lt += __shfl_xor(lt, 32);
      if (seg_open) {
        // parked (m1, l1, rows1) and this run's (m, lt, o): weights 2^(m1-M) and 2^(m-M),
        // a side whose maximum is -inf (nothing valid seen) gets weight 0 by select
        const f32x2 ml = *(const f32x2*)(rec + G * kD + 2 * n);
        const float M = fmaxf(ml.x, m);
        const float w1 = (ml.x == kNegInf) ? 0.f : __builtin_amdgcn_exp2f(ml.x - M);
        const float w2 = (m == kNegInf) ? 0.f : __builtin_amdgcn_exp2f(m - M);
        lt = w1 * ml.y + w2 * lt;
        m = M;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float keep = __shfl(w1, 4 * c + r), add = __shfl(w2, 4 * c + r);
          if (4 * c + r < G) {
#pragma unroll
            for (int t = 0; t < kTiles / 4; ++t) {
              const f32x4 p4 = *(const f32x4*)(rec + (4 * c + r) * kD + tile_group_dim<kD>(t, n));
#pragma unroll
              for (int e = 0; e < 4; ++e) o[4 * t + e][r] = keep * p4[e] + add * o[4 * t + e][r];
            }
          }
        }
      }
      if (done) {
        if (nstaged == a.staged_max) store_staged();
        staged_segs = (lane == nstaged) ? seg : staged_segs;
        uint16_t* rows = staged + nstaged * G * kD;
        const float inv = inverse(lt, a.out_scale);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int h = 4 * c + r;
          const float f = __shfl(inv, h);
          if (h < G) {
#pragma unroll
            for (int t = 0; t < kTiles / 4; ++t)
              *(u32x2*)(rows + h * kD + tile_group_dim<kD>(t, n)) =
                  finish_row4(f32x4{o[4 * t][r], o[4 * t + 1][r], o[4 * t + 2][r], o[4 * t + 3][r]}, f);
          }
        }
        ++nstaged;
        ends_flags &= ~kEndsRight;
      } else {
        if (!open_left) store_staged();   // the staged rows lie where the record goes
        ends_flags = !open_left ? ends_flags | kEndsRight
                     : (meta & kMetaSegEnd) ? kEndsLeft : kEndsLeft | kEndsThrough;
        left = open_left ? seg : left;
        right = open_left ? right : seg;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int h = 4 * c + r;
          if (h < G) {
#pragma unroll
            for (int t = 0; t < kTiles / 4; ++t)
              *(f32x4*)(rec + h * kD + tile_group_dim<kD>(t, n)) =
                  f32x4{o[4 * t][r], o[4 * t + 1][r], o[4 * t + 2][r], o[4 * t + 3][r]};
          }
        }
        if (c == 0) *(f32x2*)(rec + G * kD + 2 * n) = (n < G) ? f32x2{m, lt} : f32x2{kNegInf, 0.f};
      }
      seg_open = true;
      m = kNegInf;
      l = 0.f;
#pragma unroll
      for (int i = 0; i < kTiles; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };

  // The query group of a new (request, KV head), one block ahead of use and behind that block's KV
  // loads, so that nothing has to wait for loads younger than the ones it needs: fetched when its
  // first block was already to be consumed, it cost the pipeline a drain per segment (512 requests of
  // 16..512 tokens: 116.5 -> 114.1 us; 8 requests at D = 256: 36.3 -> 35.7).
  auto take_q = [&](int meta) {   // before the next group is asked for
    if (!(meta & kMetaSegFirst)) return;
    seg_open = false;
    seg = seg_next;
#pragma unroll
    for (int jj = 0; jj < kKSteps; ++jj) qop[jj] = (n < G) ? qnext[jj] : u32x4{0, 0, 0, 0};
  };
  // Waits for loads where it is known how many are younger.
  auto arrived_k = [](u32x4 (&k)[kKLoads]) {
#pragma unroll
    for (int jj = 0; jj < kKLoads; ++jj) asm volatile("" : : "v"(k[jj]));
  };
  auto arrived_v = [](VReg (&v)[kVLoads]) {
#pragma unroll
    for (int e = 0; e < kVLoads; ++e) asm volatile("" : : "v"(v[e]));
  };
  auto ask_q = [&](VReg (&v)[kVLoads], int j, int meta) {   // v: of the block before
    if (kWhole || !(meta & kMetaSegFirst)) return;
    if (kTwoBlocks) arrived_v(v);
    load_q(__builtin_amdgcn_readlane(dA.seg, j - jbase));
  };

  u32x4 kbuf[2][kKLoads];   // two blocks in turn, so that no buffer is ever copied
  VReg vbuf[2][kVLoads];
  Block at = block_at(0);
  issue_k(kbuf[0], at, 0, kKLoads);
  if (!kLate) issue_v(vbuf[0], at);
  if (!kWhole) load_q(__builtin_amdgcn_readlane(dA.seg, 0));
  if (wave == 0 && kLeavesWords) {
    // Word for the reduce pass, while the first loads are on their way: the segment of the workgroup's
    // last block, does it go on elsewhere?
    SharedSegment of_last = {0, 0};
    if (!whole && first_wave + kGroupWaves < W) {
      const ShareMap shares(T, W);
      const int begin = shares.start(first_wave), next = shares.start(first_wave + kGroupWaves);
      const int s = request_of(next - 1);
      const Place at = place(next - 1, s, the_request(s));
      of_last = word_of_group<kGroupWaves>(shares, blockIdx.x, begin, next, (at.s * Hkv + at.kvh) * G, next - 1 - at.b, at.nb);
    }
    if (lane == 0) word = of_last;
  }
  for (;;) {   // layers
  for (int j = 0; j < nshare; j += 2) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      u32x4 (&k)[kKLoads] = kbuf[i], (&knext)[kKLoads] = kbuf[i ^ 1];
      VReg (&v)[kVLoads] = vbuf[i], (&vnext)[kVLoads] = vbuf[i ^ 1];
      if (!kTwoBlocks) arrived_k(k);
      if (!kTwoBlocks && !kLate) arrived_v(v);
      if (!kWhole && i == 1 && j + 2 == jbase + kWindow) {   // the loads leave window A: B becomes A
        dA = dB;
        jbase += kWindow;
      }
      const Block next = block_at(j + i + 1);
      if (kLate) {
        issue_v(v, at);
        issue_k(knext, next, 0, kNextK);
      } else {
        issue_k(knext, next, 0, kKLoads);
        issue_v(vnext, next);
      }
      if (kTwoBlocks) arrived_k(k);
      if (j + i < nshare) {
        take_q(at.meta);
        ask_q(v, j + i + 1, next.meta);
        turn_k(k);
        consume(k, v, at.meta);
      }
      if (kLate) issue_k(knext, next, kNextK, kKLoads);
      at = next;
    }
    if (!kWhole && j == jbase) {   // window A has just been begun: the one after it is described now
      if (jbase + kWindow < nshare) dB = describe(jbase + kWindow);
      else dB = Window{0, 0, 0};
    }
  }
  store_staged();
  // Never: up to here the registers of the loads that went out last, behind the share's end, are their own.  As far as the compiler knows
  // they may still be on their way, and a loop of stores that took one over would wait for them in every turn, and so for the
  // acknowledgement of each hidden store.
  int never = 0;
  if (!kWhole) asm volatile("s_mov_b32 %0, 0" : "=s"(never));
  if (never) {
#pragma unroll
    for (int jj = 0; jj < kKSteps; ++jj) asm volatile("" : : "v"(qnext[jj]));
#pragma unroll
    for (int jj = 0; jj < kKLoads; ++jj) asm volatile("" : : "v"(kbuf[0][jj]));
#pragma unroll
    for (int e = 0; e < kVLoads; ++e) asm volatile("" : : "v"(vbuf[kLate][e]));
  }
  // Refused ids are reported once per wavefront, after the stream: nothing in the loop waits on it.
  if (a.id_faults && refused && lane == 0) atomicAdd(a.id_faults, refused);
  if (!kWhole) zero_empty_rows();
  uint16_t* out = layer.out;
  const bool more = kChained && of + 1 < layer_count(layers);
  const int ends = ends_flags, left_end = left;
  if (more) {
    // The next layer: its first loads are on their way while the workgroup meets (six layers of 24 requests, with a
    // workgroup of its own for each layer's range 767.9 us, this way 763.5).
    layer = layer_at(a, layers, of + 1);
    if (jbase) {   // window A is not the first one any more
      jbase = refused = 0;
      dA = describe(0);
    }
    at = block_at(0);
    issue_k(kbuf[0], at, 0, kKLoads);
    if (!kLate) issue_v(vbuf[0], at);
    load_q(__builtin_amdgcn_readlane(dA.seg, 0));
    dB = Window{0, 0, 0};
    seg_open = false;
    ends_flags = left = right = 0;
  }

  // The workgroup's merge.  Segments that meet inside the workgroup's range are finished from
  // the records in LDS.  What is left are at most two segments that it shares with other
  // workgroups: one record each goes to memory for the reduce pass, and a workgroup whose last
  // segment goes on behind it leaves word of that.
  const AttnLaunch& b = reread(a);
  const int wave_floats = b.wave_lds_floats;
  const float out_scale = b.out_scale;
  float* const records = b.ws_rec;
  asm volatile("" : : "s"(wave_floats), "s"(out_scale), "s"(records), "s"(b.ws_words));   // asked for before the meeting
  // 16 lanes have 64 floats of a segment's rows: no division by what is only known now
  const int chunks = G * (kD / 64);
  const float per_chunk = __builtin_amdgcn_rcpf((float)chunks);
  // Records asked for at a time: four where there is one chain through all wavefronts.  With that, the order above and the descriptor asked for
  // ahead, append and attention of short segments, before / after: 4 requests of 17..300 tokens on 8/2 heads 8.7 / 8.55 us, 10 of 100 in e4m3
  // at D = 64 7.3 / 7.1.  Else chains are short, 33 requests of 30..60 on 40/8 heads 11.8 / 11.8, with four 12.0.
  constexpr int kAtOnce = kWhole ? 4 : 2;
  if (!kWhole && lane == 0) {
    left_seg[wave] = left_end;
    share_ends[wave] = ends;
  }
  __syncthreads();
  if (kLeavesWords && threadIdx.x == 0) *shared_segment(b, of, blockIdx.x) = word;
  // One chain of LDS records per wavefront v whose left record ends its segment or is the
  // workgroup's last (bit v of `ending`), and one for the last wavefront's right record (bit
  // kGroupWaves).  The threads go to the chains that there are: with room for all nine, two to
  // four rounds instead of one took 1 us more (64 requests of 50..100 tokens on 40/8 heads 18.4 -> 16.6).
  // Where the workgroup has one segment, there is one chain, through all wavefronts that have blocks of it.
  int ending, through;
  if (kWhole) {
    ending = W > 1 ? 1 << last_wave : 0;
    through = (1 << last_wave) - 2;
  } else {
    const int how = lane < kGroupWaves ? share_ends[lane] : 0;
    through = (int)__ballot(how & kEndsThrough);
    ending = (int)__ballot((how & kEndsLeft) && (!(how & kEndsThrough) || lane == last_wave)) |
             (__ballot((how & kEndsRight) && lane == last_wave) ? 1 << kGroupWaves : 0);
  }
#pragma unroll 1
  for (int sub = threadIdx.x >> 4; sub < __popc(ending) * chunks; sub += kThreads / 16) {
    const int nth = (int)(((float)sub + 0.5f) * per_chunk), item = 16 * (sub - nth * chunks) + (threadIdx.x & 15);
    int rest = ending;
    for (int z = 0; z < nth; ++z) rest &= rest - 1;
    const int chain = __ffs(rest) - 1;
    const bool right_only = chain == kGroupWaves;
    const int v = right_only ? last_wave : chain;
    int u = v;
    bool from_right = true;   // the chain begins with wavefront u's right record
    if (!right_only) {
      u = 31 - __clz(~through & ((1 << v) - 1));   // the last one before v that the segment does not go through
      if (u < 0) { u = 0; from_right = false; }
    }
    const bool open_right = right_only || ((through >> v) & 1);
    const int h = item / (kD / 4);
    Partial p = kNothing;
#pragma unroll 1
    for (int k = u; k <= v; k += kAtOnce) {
      f32x2 ml[kAtOnce];
      f32x4 x[kAtOnce];
#pragma unroll
      for (int z = 0; z < kAtOnce; ++z) {
        const float* rec = wave_lds + min(k + z, v) * wave_floats + (k + z == u && from_right ? rec_floats : 0);
        ml[z] = *(const f32x2*)(rec + G * kD + 2 * h);
        x[z] = *(const f32x4*)(rec + 4 * item);
      }
#pragma unroll
      for (int z = 0; z < kAtOnce; z += 2) {   // two by two, so that every way here gives the same bits
        const f32x2 ml2[2] = {k + z > v ? f32x2{kNegInf, 0.f} : ml[z], k + z + 1 > v ? f32x2{kNegInf, 0.f} : ml[z + 1]};
        const f32x4 x2[2] = {x[z], x[z + 1]};
        fold(p, ml2, x2);
      }
    }
    if (kWhole || (from_right && !open_right)) {
      *(u32x2*)(out + (int64_t)(kWhole ? seg_next : left_seg[v]) * (G * kD) + 4 * item) = finish_row4(p.x, inverse(p.l, out_scale));
    } else {
      float* rec = group_record(b, kD, of, blockIdx.x, from_right);
      store16(rec + 4 * item, __builtin_bit_cast(u32x4, p.x));
      if (item % (kD / 4) == 0) *(f32x2*)(rec + G * kD + 2 * h) = f32x2{p.m, p.l};
    }
  }
  if (!more) return;
  ++of;
  __syncthreads();   // the records in LDS have been read
  }
}

}  // namespace
}  // namespace pkv
