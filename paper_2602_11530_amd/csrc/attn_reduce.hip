// Split-K merge for paged decode attention on gfx950: folds the records (reference max, partial
// sum, un-normalised row; the maxima are in log2 units) that the stream pass left of the segments
// (request, KV head) that several of its workgroups share into the final bf16 rows.  Segments
// that one of them holds are finished there.  Bound by latency: where the records are, then the
// records.
//
// At most one shared segment begins in a workgroup of the stream pass, whose
// wavefronts have met in LDS: one workgroup here for each there (256), which reads one word and is done when
// no segment goes on behind that one's range.  A segment of more than a few records has the workgroups of its middle, too.
#include "attn_partial.h"
#include "pkv_kernels.h"

namespace pkv {
namespace {

constexpr int kBatch = 4;   // records in flight per thread

// A segment that workgroups of the stream pass share.  16 lanes have a chunk of 64 floats of its rows, so that what a thread does
// follows from shifts, and offsets are 32-bit.  With 16 bytes to each thread in order, divisions, 64-bit products and eight loads unrolled,
// 0.85 us passed between the word and the last load going out (time stamps), as long as the loads and the folding take together;
// 33 records took two turns.  Append and attention, before / this way: one request of 8191 tokens 16.2 / 15.5 us, 8 at D = 256
// 32.6 / 32.1, 512 of 16..512 106.1 / 104.0, 32 at D = 64 43.2 / 41.9, 64 of 1024..8192 194.3 / 192.7, on 8-bit pools 104.3 / 102.9,
// six layers of 24 754 / 747.
//   Up to kBatch records, or twice that: a thread loads all of them at once and is done.  From kBatch + 1 to twice as many by several
//   workgroups and sets of lanes, as below: 8 requests of 1500..3000 tokens on 32/8 heads at D = 64 15.8 us, this way 15.0, 8 at
//   D = 256 31.5 / 30.8; with four times kBatch at once 0 to 1 % slower than below.
//   More: the workgroups in the middle of the segment, in which nothing begins, take some of the chunks each, and in a workgroup
//   sets of lanes take every sets-th record and meet in LDS, four to one at a time.
template <int kD>
struct SegmentRecords {
  const char* base;    // the segment's first record
  uint32_t rec_bytes;
  uint32_t at, stats;  // of this lane's 16 bytes, and of its head's statistics, within a record
  // kN records i, i + step, ... of `count`: those past the end are the last one with nothing valid
  template <int kN>
  __device__ __forceinline__ void fold_batch(Partial& p, int i, int step, int count) const {
    f32x4 x[kN];
    f32x2 ml[kN];
#pragma unroll
    for (int z = 0; z < kN; ++z) {
      const int j = min(i + z * step, count - 1);
      // the one that begins the segment is its workgroup's second record, the others are first ones
      const uint32_t off = (uint32_t)(2 * j - (j > 0)) * rec_bytes;
      x[z] = *(const f32x4*)(base + (off + at));
      ml[z] = *(const f32x2*)(base + (off + stats));
    }
#pragma unroll
    for (int z = 0; z < kN; ++z) {
      if (i + z * step >= count) ml[z].x = kNegInf;
    }
    fold(p, ml, x);
  }
};
template <int kD, typename Layers>
__device__ __forceinline__ void reduce_segment(const AttnLaunch& a, const Layers& layers, const SharedSegment& seg, int group) {
  constexpr int kHeadChunks = kD / 64;
  const int sub = threadIdx.x >> 4, lane16 = threadIdx.x & 15;
  const int chunks = a.G * kHeadChunks, count = seg.records(), slice = seg.slice();
  uint16_t* out = layer_of(a, layers).out + (int64_t)seg.row * kD;
  SegmentRecords<kD> r;
  r.base = (const char*)group_record(a, kD, layer_index(layers), group - slice, true);
  r.rec_bytes = record_floats(a.G, kD) * (uint32_t)sizeof(float);
  auto place = [&](int chunk) {
    r.at = 256 * chunk + 16 * lane16;
    r.stats = 4 * a.G * kD + 8 * (chunk / kHeadChunks);
  };
  auto finish = [&](const Partial& p, int chunk) {
    *(u32x2*)(out + 64 * chunk + 4 * lane16) = finish_row4(p.x, inverse(p.l, a.out_scale));
  };
  if (count <= 2 * kBatch) {
    if (slice != 0 || sub >= chunks) return;
    place(sub);
    Partial p = kNothing;
    if (__builtin_expect(count <= kBatch, 1)) r.template fold_batch<kBatch>(p, 0, 1, count);
    else r.template fold_batch<2 * kBatch>(p, 0, 1, count);
    finish(p, sub);
    return;
  }
  __shared__ f32x4 rows[kReduceThreads];
  __shared__ f32x2 stats[kReduceThreads];
  const RecordSplit split(count, chunks);
  const int mine = split.mine;
  if (slice * mine >= chunks) return;
  int sets = split.sets;
  const int set = split.quotient(sub, mine), chunk = slice * mine + (sub - set * mine);
  const bool works = set < sets && chunk < chunks;
  Partial p = kNothing;
  if (works) {
    place(chunk);
    for (int i = set; i < count; i += kBatch * sets) r.template fold_batch<kBatch>(p, i, sets, count);
  }
  while (sets > 1) {
    rows[threadIdx.x] = p.x;
    stats[threadIdx.x] = f32x2{p.m, p.l};
    __syncthreads();
    const int left = (sets + 3) >> 2;
    if (set < left) {
      f32x4 x[3];
      f32x2 ml[3];
#pragma unroll
      for (int z = 0; z < 3; ++z) {
        const bool there = set + (z + 1) * left < sets;
        const int t = threadIdx.x + (there ? (z + 1) * left * mine * 16 : 0);
        x[z] = rows[t];
        ml[z] = stats[t];
        if (!there) ml[z].x = kNegInf;
      }
      fold(p, ml, x);
    }
    sets = left;
    __syncthreads();
  }
  if (works && set == 0) finish(p, chunk);
}

// The word of this workgroup.  What follows it needs of the launch descriptor is asked for before it: the descriptor is several cache
// lines, each a round trip of its own.
template <typename Layers>
__device__ __forceinline__ SharedSegment read_word(const AttnLaunch& a, const Layers& layers) {
  asm volatile("" : : "s"(a.ws_words), "s"(a.ws_rec), "s"(a.G), "s"(a.out_scale), "s"(layer_of(a, layers).out));
  return *shared_segment(a, layer_index(layers), blockIdx.x);
}
template <int kD, typename Layers>
__global__ __launch_bounds__(kReduceThreads) void attn_reduce_group_kernel(AttnLaunch a, Layers layers) {
  const SharedSegment seg = read_word(a, layers);
  if (seg.told > 0) reduce_segment<kD>(a, layers, seg, blockIdx.x);
}

}  // namespace

template <int kD>
static void launch_dim(const AttnLaunch& a, const AttnLayers* layers, dim3 groups, hipStream_t stream) {
  if (layers) hipLaunchKernelGGL((attn_reduce_group_kernel<kD, AttnLayers>), groups, dim3(kReduceThreads), 0, stream, a, *layers);
  else hipLaunchKernelGGL((attn_reduce_group_kernel<kD, OneLayer>), groups, dim3(kReduceThreads), 0, stream, a, OneLayer{});
}

hipError_t launch_attn_reduce(const AttnLaunch& a, const AttnLayers* layers, hipStream_t stream) {
  const dim3 groups(a.waves / group_waves(a.D), layers ? layers->count : 1);
  if (a.D == 64) launch_dim<64>(a, layers, groups, stream);
  else if (a.D == 128) launch_dim<128>(a, layers, groups, stream);
  else if (a.D == 256) launch_dim<256>(a, layers, groups, stream);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace pkv
