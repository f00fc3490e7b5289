// Internal launch interface between the C-ABI layer and the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace pkv {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));  // one 16-byte lane load

constexpr int kBlockTokens = 16;     // tokens per streaming unit (one MFMA tile of keys); a physical
                                     // block of B = 16, 32 or 64 tokens holds B/16 units per KV head
constexpr int kMaxBlockSize = 64;
constexpr int kMaxPartition = 65536; // tokens covered by one partial result, upper bound
constexpr int kMaxGroup = 16;        // query heads per KV head
constexpr int kMaxSeqs = 2048;       // per-request prefix arrays live in LDS

// The attention pass is a persistent launch sized for the 256 compute units of
// an MI355X: one workgroup per unit, of two wavefronts per SIMD (one at D = 256, where a
// wavefront needs most of a SIMD's registers), each streaming an equal share of the batch's KV
// blocks.
constexpr int kLayerGroups = 256;   // workgroups per layer of the attention pass
constexpr int kStreamWaves = 8 * kLayerGroups;
// Wavefronts per workgroup.
__host__ __device__ constexpr int group_waves(int D) { return D == 256 ? 4 : 8; }

// Stream pass where V goes out when K is there: K loads, of four (D = 128) or eight, of the next block that go out with this
// block's V.  All four where shares are short (short_at_128).
constexpr int kAhead = 2;

// How the batch's KV blocks are laid out as one stream and cut into shares.
//   Segment (s, kvh) holds the nblk_s = ceil(L_s/16) 16-token units ("blocks" below;
//   a physical block of B tokens is B/16 of them in a row) of request s for KV
//   head kvh; segments follow each other in (s, kvh) order; position pos of the
//   stream is block b of segment (s, kvh) with
//       pos = Hkv * cumB[s] + kvh * nblk_s + b,     cumB[s] = sum_{s'<s} nblk_s'.
//   Wavefront w owns positions [w*T/W, (w+1)*T/W), T = Hkv * cumB[S].
//   A run is a maximal stretch of one wavefront's share inside one segment and
//   one partition (P tokens of the request); every run yields one partial result
//   (max, sum, un-normalised row) per query head of the group.  The runs of one
//   segment inside one share are folded together.  A segment that lies wholly
//   inside a share is finished there; of any other the wavefront leaves a record
//   in LDS.  The wavefronts of a workgroup fold those, finish the segments that lie
//   inside the workgroup's range and leave one record in memory for each of the two segments
//   that may cross its ends (group_record); the workgroup in which a crossing segment
//   begins, and those that lie in the middle of one, leave word of it (SharedSegment).
//
// Shares begin at floor(w * T / W), so that the longer ones are spread evenly over the compute
// units: with the longer ones first, the units that hold them end last (1.5 % on 64 requests of
// 1024..8192 tokens, whose shares have 70 and 71 blocks).  In 32 bits and without divisions, because both functions
// sit on short critical chains: W is a power of two, as a full launch's and a workgroup's are, or T.
struct ShareMap {
  uint32_t T, W, shift, len, more;   // more of the W shares have len + 1 positions
  __host__ __device__ ShareMap(uint32_t T_, uint32_t W_) : T(T_), W(W_) {
    const bool even = (W & (W - 1)) == 0;
    shift = even ? __builtin_ctz(W) : 0;
    len = even ? T >> shift : 1;
    more = T - len * W;
  }
  __host__ __device__ uint32_t start(uint32_t w) const { return w * len + ((w * more) >> shift); }   // W <= 2^16
  // The wavefront whose share holds position pos: an estimate that is off by less than one, put right.
  __host__ __device__ uint32_t owner(uint32_t pos) const {
    uint32_t w = (uint32_t)((float)pos * ((float)W / (float)T));
    w = w < W ? w : W - 1;
    const uint32_t at = start(w), next = start(w + 1);
    return at > pos ? w - 1 : next <= pos ? w + 1 : w;
  }
};
__host__ __device__ inline int64_t share_start(int64_t w, int64_t T, int64_t W) {
  return ShareMap((uint32_t)T, (uint32_t)W).start((uint32_t)w);
}
__host__ __device__ inline int share_owner(int64_t pos, int64_t T, int64_t W) {
  return (int)ShareMap((uint32_t)T, (uint32_t)W).owner((uint32_t)pos);
}
// Wavefronts that take part.
__host__ __device__ inline int share_count(int T, int waves) { return T < waves ? T : waves; }

// One partial record: G un-normalised rows of D floats, then (reference max in
// log2 units, partial sum) for up to kMaxGroup heads.  Rows are 16-byte multiples.
__host__ __device__ inline int record_floats(int G, int D) { return G * D + 2 * kMaxGroup; }

// A batch with no more segments than the launch has workgroups, none longer than this many blocks, is cut
// along the segments.  Up to 6 blocks per wavefront; with at most 64 of them, which leave most
// compute units idle, 3 where a block is 8 KiB or more.  Cut along the segments / not, us for append and
// attention: 8 segments of 40/8 heads at D = 128, 384 tokens (3 blocks) 13.2 / 13.4, 512 13.2 / 12.8, 768
// 17.3 / 13.7; 16 segments of 8/1 heads, 768 tokens 20.0 / 15.5; 128 of 40/8 heads, 512 17.6 / 18.8, 768
// 21.4 / 21.7; 240, 768 23.5 / 27.7; blocks of 4 KiB (D = 64), 8 segments of 768 tokens 12.2 / 13.0.
inline int short_segment(int64_t segments, int D, bool kv_fp8) {
  const int block_bytes = 2 * kBlockTokens * D * (kv_fp8 ? 1 : 2);
  return (segments <= 64 && block_bytes >= 8192 ? 3 : 6) * group_waves(D);
}

// A segment that several workgroups share, as those of them leave it in which no later one begins: the one that it begins in and
// those in its middle.
struct SharedSegment {
  int row;    // first output row
  int told;   // workgroups that share it, and from bit 16 how many of them come before this one; 0 when there is none
  __host__ __device__ int records() const { return told & 0xffff; }
  __host__ __device__ int slice() const { return told >> 16; }
};
// The word of workgroup `group` of a batch of workgroups' records, which has positions `from` to `next` of the stream: its last block's
// segment has `blocks` of them from position `begin` on, and `row` is its first output row.
template <int kGroupWaves>
__host__ __device__ __forceinline__ SharedSegment word_of_group(const ShareMap& shares, int group, int from, int next, int row, int begin,
                                                                int blocks) {
  SharedSegment w = {0, 0};
  if (begin + blocks > next) {
    const int first = begin >= from ? group : (int)shares.owner(begin) / kGroupWaves;
    w.row = row;
    w.told = ((int)shares.owner(begin + blocks - 1) / kGroupWaves - first + 1) | (group - first) << 16;
  }
  return w;
}

// How the workgroups that leave word of a segment share its records in the reduce pass, where it has more than a thread loads at once: each
// has `mine` chunks of 64 floats of the rows, 16 lanes to a chunk, and `sets` of lanes a chunk's records in turn.
constexpr int kReduceThreads = 512;
constexpr int kReduceSubs = kReduceThreads / 16;   // G * D / 64 is kReduceSubs at most
struct RecordSplit {
  int mine, sets;
  // small quotients by way of fp32: (x + 1/2) / n is at least 1 / (2n) away from a whole number
  __host__ __device__ static int quotient(int x, int n) {
#ifdef __HIP_DEVICE_COMPILE__
    const float per = __builtin_amdgcn_rcpf((float)n);
#else
    const float per = 1.f / (float)n;
#endif
    return (int)(((float)x + 0.5f) * per);
  }
  __host__ __device__ RecordSplit(int count, int chunks) {
    const int helpers = count - 1 < chunks ? count - 1 : chunks;
    mine = quotient(chunks + helpers - 1, helpers);
    sets = quotient(kReduceSubs, mine);
    sets = sets < count ? sets : count;
  }
};

// What differs between the layers of one launch.
struct AttnLayer {
  const uint16_t* q;
  const void* k_pool;   // bf16, or e4m3 bytes when kv_fp8
  const void* v_pool;
  uint16_t* out;
};
constexpr int kMaxLaunchLayers = 8;

struct AttnLaunch {
  AttnLayer layer;
  const int32_t* block_tables;
  const int32_t* context_lens;
  float* ws_rec;   // the first layer's partial records, see group_record()
  float* ws_words; // and SharedSegments
  int leaves_records;  // 0: the bounds alone say that each segment has a workgroup, none is shared, and there is no reduce pass
  int short_blocks;    // see short_segment()
  float scale_log2e;   // softmax scale x log2(e) (x the K pool's scale for an e4m3 pool)
  float out_scale;     // applied to the normalised row: 1, or the V pool's scale
  int kv_fp8;          // the pools hold one-byte e4m3 values
  int32_t* id_faults;  // optional device counter of refused block ids (nullptr: not reported)
  int S, Hq, Hkv, G, MAXB;
  int D;           // head dimension: 64, 128 or 256
  int waves;       // persistent wavefronts of the stream pass: kStreamWaves, or half of it for D = 256
  int upb;         // 16-token units per physical block (B / 16)
  int P;           // partition size, tokens
  int max_ctx;     // context lengths are clamped to [0, max_ctx] (<= MAXB * 16)
  int NB;          // physical blocks per pool; ids outside [0, NB) are never followed
  int wave_lds_floats;  // a wavefront's share of LDS: its left record, then its right record or staged rows
  int staged_max;       // finished segments whose rows a wavefront can stage in LDS
  int turns;            // there is room in LDS to turn K
  int64_t layer_ws_floats;   // workspace from one layer's records to the next one's
};
// The layers of a launch, blockIdx.y being the layer.  A second kernel argument, so that a launch of one layer reads its pointers
// with the rest (the look-up costs one request of 8191 tokens 0.4 us).
struct AttnLayers {
  int count;
  AttnLayer layer[kMaxLaunchLayers];
};
struct OneLayer {};
struct WholeLayer : OneLayer {};   // a workgroup for each segment
// One after the other in each workgroup.
struct ChainedLayers : AttnLayers {};
__device__ __forceinline__ int layer_index(const OneLayer&) { return 0; }
__device__ __forceinline__ int layer_index(const AttnLayers&) { return blockIdx.y; }
__device__ __forceinline__ int layer_index(const ChainedLayers&) { return 0; }
__device__ __forceinline__ int layer_count(const OneLayer&) { return 1; }
__device__ __forceinline__ int layer_count(const AttnLayers& l) { return l.count; }
__device__ __forceinline__ const AttnLayer& layer_at(const AttnLaunch& a, const OneLayer&, int) { return a.layer; }
__device__ __forceinline__ const AttnLayer& layer_at(const AttnLaunch&, const AttnLayers& l, int i) { return l.layer[i]; }
__device__ __forceinline__ const AttnLayer& layer_of(const AttnLaunch& a, const OneLayer&) { return a.layer; }
__device__ __forceinline__ const AttnLayer& layer_of(const AttnLaunch&, const AttnLayers& l) { return l.layer[layer_index(l)]; }

// The workspace, per layer: two records per workgroup of the stream pass (of the shared segment that begins in
// it, and of the one that begins in an earlier one), then each workgroup's SharedSegment.
__host__ __device__ inline float* group_record(const AttnLaunch& a, int D, int layer, int group, bool begins_here) {
  return a.ws_rec + layer * a.layer_ws_floats + (int64_t)(2 * group + begins_here) * record_floats(a.G, D);
}
__host__ __device__ inline SharedSegment* shared_segment(const AttnLaunch& a, int layer, int group) {
  return (SharedSegment*)(a.ws_words + layer * a.layer_ws_floats) + group;
}
constexpr int kRecordsBeforeWords = 2 * kLayerGroups;
// Per layer: a whole number of records, so that every layer's are aligned like the first one's.
__host__ __device__ inline int64_t layer_ws_floats(int G, int D) {
  const int64_t rec = record_floats(G, D), words = kLayerGroups * (int64_t)sizeof(SharedSegment) / sizeof(float);
  return kRecordsBeforeWords * rec + (words + rec - 1) / rec * rec;
}

// LDS of a workgroup of the stream pass, in floats: the prefix arrays, then per wavefront a left record
// and room for a right record or up to 8 finished segments' rows, held to 78 KiB.  One workgroup takes a
// CU's registers, so LDS would allow twice that, but 8 staged segments instead of 5 (G = 5, D = 128) gain
// nothing: 512 requests of 16..512 tokens 110.2 us at 78 KiB, 112.2 at 152; 64 of 1024..8192 190.7 and 189.2.
// Records and rows are read and written 16 bytes at a time and lie on 16-byte boundaries; 4-byte ones,
// which the LDS unit also accepts, cost those 512 requests 1.6 us and 4 of 17..300 tokens 0.3 of 12.4.
struct StreamLds {
  int prefix, wave;   // where the wavefronts' parts begin, and from one to the next
  int staged_max;
  int bytes;
  int turn_bytes;     // behind them, a block of K per wavefront, to turn it; 0 where there is no room or no need
};
inline StreamLds stream_lds(int S, int G, int D, bool kv_fp8 = false) {
  const int group = group_waves(D), rec = record_floats(G, D), rows = G * D / 2;
  StreamLds l;
  l.prefix = (2 * (S + 1) + 3) & ~3;
  const int budget = ((78 * 256 - l.prefix) / group - rec) & ~3;
  int room = budget < 8 * rows ? budget : 8 * rows;
  if (room < rec) room = rec;
  l.wave = rec + room;
  l.staged_max = room / rows;
  l.bytes = (l.prefix + group * l.wave) * (int)sizeof(float);
  // Two whole records per wavefront come first: at D = 128 there is no room for K with 16 query heads per KV head, in bf16
  // with 15 from 640 requests and with 14 from 1664; in e4m3 with 16 from 1664.
  l.turn_bytes = group * kBlockTokens * D * (kv_fp8 ? 1 : 2);
  if (l.bytes + l.turn_bytes > 159 * 1024 || (D == 64 && kv_fp8)) l.turn_bytes = 0;
  return l;
}

// D = 256: does a batch take the kernel for large ones?  Where the bounds allow shares of 24 blocks and more.  Us for append and
// attention, small / large:
//   bf16: V goes out a block ahead / when K is there, with a quarter of the next K.  20 requests of 260..350 tokens on 8/8 heads (3
//       blocks a share) 16.6 / 18.4, 20 of 350..470 (4) 22.2 / 22.4, 20 of 700..940 (8) 32.7 / 32.8; 20 of 2600..3500 (30) 86.1 /
//       85.5, 20 of 6100..8200 (70) 191.7 / 186.8, 125 of 970..1320 on 40/8 heads (70) 196.9 / 192.2.  (With K loaded in operand
//       order and two blocks out the last three took 87.4, 188.9 and 194.)  Both loops in one kernel cost it 75 registers and
//       short shares 5 to 14 %.
//   e4m3: K turned in LDS / loaded in operand order.  20 of 85..120 on 8/8 heads (1) 11.0 / 11.5; shares of 2 to 16 blocks 0.4 %
//       either way; 20 of 6100..8200 on 40/8 heads (70) 108.3 / 104.8, 600 of 2800..3750 on 8/1 heads (120) 173.4 / 170.3.  Both
//       in one kernel cost short shares 1 to 3 %.
inline bool large_at_256(const AttnLaunch& a) {
  const int64_t most = (int64_t)a.S * a.Hkv * ((a.max_ctx + kBlockTokens - 1) / kBlockTokens);
  return a.D == 256 && most >= 24 * (int64_t)a.waves;
}
// D = 128 in bf16: does a batch take the kernel for short shares?  There all of the next block's K goes out with this block's V and a
// wavefront waits for loads once a block; else half of it, see attn_stream.h.  Up to 16 blocks a share by the bounds, which are
// often twice the mean.  All / half, append and attention, geometric means of 16 shapes each (8 to 600 segments, 1 to 8 heads per
// KV head): shares of 1 block 0.979, 2 0.966, 3 0.963, 4 0.978, 6 0.985, 8 0.989, 12 0.998, 20 1.002; 70 blocks 1.01.  A choice
// within one kernel costs what it gains (a second loop: 4 requests of 17..300 tokens 10.9 -> 11.25 us).
inline bool short_at_128(const AttnLaunch& a) {
  const int64_t most = (int64_t)a.S * a.Hkv * ((a.max_ctx + kBlockTokens - 1) / kBlockTokens);
  return a.D == 128 && !a.kv_fp8 && most <= 16 * (int64_t)a.waves;
}
// The stream pass's kernels for one layer of those, and for layers one after the other.
void launch_large_256(const AttnLaunch& a, size_t lds, hipStream_t stream);
void launch_short_128(const AttnLaunch& a, size_t lds, hipStream_t stream);
void launch_whole(const AttnLaunch& a, size_t lds, hipStream_t stream);
void launch_chained_short_128(const AttnLaunch& a, const AttnLayers& layers, size_t lds, hipStream_t stream);
hipError_t launch_chained(const AttnLaunch& a, const AttnLayers& layers, size_t lds, hipStream_t stream);

// The turn of a block of K: place, in 16-byte pieces, of piece p of token t (`pieces` of them each: 8, 16 or 32).  A wavefront writes
// 64 pieces in a row and reads, lane 16*c + n, piece 4*jj + c of token turn_token(n).  The LDS unit takes a read of 16 bytes a
// lane in four steps of 16 lanes over 64 banks, and a step has lanes of two c (0..3, 12..15 and 20..27; 4..11, 16..19 and 28..31;
// the same of the upper half); a write in eight steps of 8 lanes in a row over 32 banks.  Here the tokens of a
// step, all different, differ in the bits of the place that c does not reach: no conflicts either way.  With t itself for a key
// every read took 8 steps instead of 4 (SQ_LDS_BANK_CONFLICT, profiles/attn_stream_lds.md).
__host__ __device__ constexpr int turn_token(int n) { return 4 * (n & 3) + (n >> 2); }
__host__ __device__ constexpr int turn_place(int pieces, int t, int p) {
  return t * pieces + (p ^ (pieces == 8 ? (t >> 2) | (t & 2) << 1 : (t >> 2) | (t & 3) << 2));
}

// Stream pass: persistent wavefronts, which finish what they have to themselves and leave records of the rest.
// `layers`: nullptr for the one layer of `a`.
hipError_t launch_attn_stream(const AttnLaunch& a, const AttnLayers* layers, hipStream_t stream);
// Reduce pass: the segments that several workgroups share, from their records.
hipError_t launch_attn_reduce(const AttnLaunch& a, const AttnLayers* layers, hipStream_t stream);

// Plain device-to-device copy.
hipError_t launch_copy(const void* src, void* dst, int64_t bytes, hipStream_t stream);

// Whole-block copies; `gather` selects the direction.
// `id_faults` (optional, device): incremented once per listed block that is skipped because an
// id lies outside its pool.
hipError_t launch_kv_block_copy(const void* src, void* dst, const int32_t* block_ids,
                                int64_t n_blocks, int64_t block_bytes, int64_t num_pool_blocks,
                                bool gather, int32_t* id_faults, hipStream_t stream);

// Pool to pool: dst[dst_ids[i]] = src[src_ids[i]], no staging image in between.
hipError_t launch_kv_block_move(const void* src, const int32_t* src_ids, int64_t src_pool_blocks,
                                void* dst, const int32_t* dst_ids, int64_t dst_pool_blocks,
                                int64_t n_blocks, int64_t block_bytes, int32_t* id_faults,
                                hipStream_t stream);

// New token's K and V rows into slot context_lens[s] - 1 of every request.
hipError_t launch_kv_append(const uint16_t* k_new, const uint16_t* v_new, uint16_t* k_pool,
                            uint16_t* v_pool, const int32_t* block_tables,
                            const int32_t* context_lens, int S, int Hkv, int D, int MAXB, int B,
                            int max_ctx, int NB, int32_t* id_faults, hipStream_t stream);

// The same for one-byte E4M3 pools: rows are divided by the pool's scale and rounded to E4M3.
hipError_t launch_kv_append_fp8(const uint16_t* k_new, const uint16_t* v_new, void* k_pool,
                                void* v_pool, const int32_t* block_tables,
                                const int32_t* context_lens, float k_scale, float v_scale, int S,
                                int Hkv, int D, int MAXB, int B, int max_ctx, int NB,
                                int32_t* id_faults, hipStream_t stream);

// Measurement aid: the stream pass's loads at D = 128 in bf16 with no arithmetic (see stream_probe.hip).
hipError_t launch_stream_read_probe(const void* k_buf, const void* v_buf, uint32_t num_slabs,
                                    int64_t total_blocks, void* sink, hipStream_t stream);

}  // namespace pkv
