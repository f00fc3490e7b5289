// Split-K merge for paged decode attention on gfx950: folds the records (reference max, partial
// sum, un-normalised row; the maxima are in log2 units) that the stream pass left of the segments
// (request, KV head) that several of its wavefronts share into the final bf16 rows.  Segments
// that one share holds are finished there.  Bound by latency: where the records are, then the
// records.  Two layouts (pkv_kernels.h):
//
// Records of workgroups: at most one shared segment begins in a workgroup of the stream pass, whose
// wavefronts have met in LDS: one workgroup here for each there (256), which reads one word and is done when
// no segment goes on behind that one's range.  A segment of more than a few records has the workgroups of its middle, too.
//
// Records of wavefronts (by rows), as they come: a workgroup for each row fetches the statistics side by side and
// then streams the partial rows sixteen at a time.
#include "attn_partial.h"
#include "pkv_kernels.h"

namespace pkv {
namespace {

constexpr int kBatch = 4;      // records in flight per thread
constexpr int kRowBatch = 16;  // partial rows in flight per wavefront, by rows

constexpr int kRow = 64;       // floats of a row of a batch that goes by rows (what_is_left): one per lane

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o));
  return x;
}
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
  return x;
}

// Where the records of row (s, h) lie: the slots of its segment's first and last
// block's owners (see pkv_kernels.h).  Returns false when there is nothing to fold: an empty
// request, a segment that one wavefront finished, a batch that did not go by rows (cumB[0] < 0).
struct RowRecords {
  int first;   // slot of the first record
  int np;      // one record per wavefront that streamed part of this segment
  int g;       // head within its KV head's group
};
__device__ __forceinline__ bool locate_records(const AttnLaunch& a, int row, RowRecords& r) {
  const int s = row / a.Hq, h = row - s * a.Hq;
  const int kvh = h / a.G;
  r.g = h - kvh * a.G;
  const int* cumB = a.ws_cum;
  const int nb = cumB[s + 1] - cumB[s];
  if (nb <= 0 || cumB[0] < 0) return false;
  const int T = a.Hkv * cumB[a.S];
  const ShareMap shares(T, share_count(T, a.waves));
  const int pos_a = a.Hkv * cumB[s] + kvh * nb;   // the segment's first block
  const int seg = s * a.Hkv + kvh, first = shares.owner(pos_a);
  r.first = seg + first;
  r.np = shares.owner(pos_a + nb - 1) - first + 1;
  return r.np > 1;
}

// One wavefront folds `count` records of a row (records begin, begin + stride, ...
// counted from the row's first): on return M is their largest reference maximum,
// acc this lane's float of the sum of their rows weighted by 2^(m - M), and
// lsum the wave-wide sum of their partial sums with the same weights.  count = 0
// leaves (M, lsum, acc) = (-inf, 0, 0).
__device__ __forceinline__ void fold_records(const AttnLaunch& a, const RowRecords& r, int begin,
                                             int stride, int count, int lane, float& M, float& lsum, float& acc) {
  const int rec_floats = record_floats(a.G, kRow);
  auto record = [&](int i) -> const float* {
    return a.ws_rec + (int64_t)(r.first + begin + i * stride) * rec_floats;
  };
  auto stats = [&](int i) -> float2 {   // (max, sum) of record i for this head
    return *(const float2*)(record(i) + a.G * kRow + 2 * r.g);
  };
  // the statistics of the first 64 records stay in registers for the second pass
  const float2 ml0 = (lane < count) ? stats(lane) : float2{kNegInf, 0.f};
  M = ml0.x;
  for (int i0 = 64; i0 < count; i0 += 64) {
    const int i = i0 + lane;
    if (i < count) M = fmaxf(M, stats(i).x);
  }
  M = wave_max(M);

  lsum = acc = 0.f;
  for (int i0 = 0; i0 < count; i0 += 64) {
    const int i = i0 + lane;
    float w = 0.f;
    if (i < count) {
      const float2 ml = i0 == 0 ? ml0 : stats(i);
      // A record whose blocks were all unmapped carries max = -inf, sum = 0.
      w = (ml.x == kNegInf) ? 0.f : __builtin_amdgcn_exp2f(ml.x - M);
      lsum = __builtin_fmaf(w, ml.y, lsum);
    }
    const int cnt = min(64, count - i0);
    for (int j0 = 0; j0 < cnt; j0 += kRowBatch) {
      float v[kRowBatch], wj[kRowBatch];
#pragma unroll
      for (int u = 0; u < kRowBatch; ++u) {
        const int j = min(j0 + u, cnt - 1);   // clamped rows get weight 0
        wj[u] = (j0 + u < cnt) ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), j)) : 0.f;
        v[u] = record(i0 + j)[r.g * kRow + lane];
      }
#pragma unroll
      for (int u = 0; u < kRowBatch; ++u)   // a weight of exactly zero must also silence whatever the row holds
        acc = (wj[u] != 0.f) ? __builtin_fmaf(wj[u], v[u], acc) : acc;
    }
  }
  lsum = wave_sum(lsum);
}

// A row of a batch that goes by rows.  Wavefront i of the workgroup folds records i, i + n, i + 2n, ...
// (n = wavefronts in the workgroup), the partial results meet in LDS and wavefront 0 folds those, normalises, scales and rounds once
// to bf16.
__device__ __forceinline__ void reduce_row(const AttnLaunch& a, int row) {
  constexpr int kWidth = kReduceThreads / 64;
  __shared__ float part_stats[kWidth][2];
  __shared__ float part_acc[kWidth][kRow];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  RowRecords r;
  if (!locate_records(a, row, r)) return;   // the same for every wavefront of the workgroup
  float M, lsum, acc;
  const int count = r.np > wave ? (r.np - wave + kWidth - 1) / kWidth : 0;
  fold_records(a, r, wave, kWidth, count, lane, M, lsum, acc);
  if (lane == 0) { part_stats[wave][0] = M; part_stats[wave][1] = lsum; }
  part_acc[wave][lane] = acc;
  __syncthreads();
  if (wave == 0) {
    float Mall = kNegInf;
    for (int w = 0; w < kWidth; ++w) Mall = fmaxf(Mall, part_stats[w][0]);
    float lall = 0.f, total = 0.f;
    for (int w = 0; w < kWidth; ++w) {
      const float m = part_stats[w][0];
      if (m == kNegInf) continue;   // nothing valid behind this partial result: weight 0
      const float f = __builtin_amdgcn_exp2f(m - Mall);
      lall = __builtin_fmaf(f, part_stats[w][1], lall);
      total = __builtin_fmaf(f, part_acc[w][lane], total);
    }
    a.layer.out[(int64_t)row * kRow + lane] = (uint16_t)pack_bf16(total * inverse(lall, a.out_scale), 0.f);
  }
  __syncthreads();   // the next row uses the same LDS
}
__device__ __forceinline__ void reduce_rows(const AttnLaunch& a) {
  for (int row = blockIdx.x; row < a.S * a.Hq; row += gridDim.x) reduce_row(a, row);
}

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
// Many segments.
template <int kD, typename Layers>
__global__ __launch_bounds__(kReduceThreads) void attn_reduce_group_kernel(AttnLaunch a, Layers layers) {
  const SharedSegment seg = read_word(a, layers);
  if (seg.told > 0) reduce_segment<kD>(a, layers, seg, blockIdx.x);
}
// Few segments: whichever of the two the stream pass has chosen, as the first prefix sum says.  That and the word are asked for together (one
// after the other 0.2 us more: 8 requests of 1500..4000 tokens on 8/8 heads at D = 64 16.4 / 16.9).
__global__ __launch_bounds__(kReduceThreads) void attn_reduce_few_kernel(AttnLaunch a) {
  asm volatile("" : : "s"(a.ws_cum), "s"(a.ws_words), "s"(a.ws_rec), "s"(a.G), "s"(a.out_scale), "s"(a.layer.out));
  const int first = a.ws_cum[0];
  const SharedSegment seg = *shared_segment(a, 0, blockIdx.x);
  asm volatile("" : : "v"(first), "v"(seg.told), "v"(seg.row));
  if (first >= 0) reduce_rows(a);   // by rows: there records may lie over the words
  else if (seg.told > 0) reduce_segment<kRow>(a, OneLayer{}, seg, blockIdx.x);
}
__global__ __launch_bounds__(kReduceThreads) void attn_reduce_rows_kernel(AttnLaunch a) {
  reduce_rows(a);
}

}  // namespace

template <int kD>
static void launch_dim(const AttnLaunch& a, const AttnLayers* layers, dim3 groups, hipStream_t stream) {
  if (layers) hipLaunchKernelGGL((attn_reduce_group_kernel<kD, AttnLayers>), groups, dim3(kReduceThreads), 0, stream, a, *layers);
  else hipLaunchKernelGGL((attn_reduce_group_kernel<kD, OneLayer>), groups, dim3(kReduceThreads), 0, stream, a, OneLayer{});
}

hipError_t launch_attn_reduce(const AttnLaunch& a, const AttnLayers* layers, hipStream_t stream) {
  const dim3 groups(a.waves / group_waves(a.D), layers ? layers->count : 1), block(kReduceThreads);
  if (a.leaves != kManySegments && (layers || a.D != kRow)) return hipErrorInvalidValue;   // one layer has the whole workspace
  if (a.leaves == kRows) hipLaunchKernelGGL(attn_reduce_rows_kernel, dim3(a.S * a.Hq), block, 0, stream, a);
  else if (a.leaves == kFewSegments) hipLaunchKernelGGL(attn_reduce_few_kernel, groups, block, 0, stream, a);
  else if (a.D == 64) launch_dim<64>(a, layers, groups, stream);
  else if (a.D == 128) launch_dim<128>(a, layers, groups, stream);
  else if (a.D == 256) launch_dim<256>(a, layers, groups, stream);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace pkv
