// Split-K merge for paged decode attention on gfx950: folds the records (reference max, partial
// sum, un-normalised row; the maxima are in log2 units) that the stream pass left of the segments
// (request, KV head) that several of its wavefronts share into the final bf16 rows.  Segments
// that one share holds are finished there.  Bound by latency: where the records are, then the
// records.  Two layouts (pkv_kernels.h):
//
// Records of workgroups: at most one shared segment begins in a workgroup of the stream pass, whose
// wavefronts have met in LDS, so that a segment has a handful of records: one workgroup
// here for each there (256), which reads one word and is done when nothing begins there.
//
// Records of wavefronts (by rows): up to hundreds of a segment, as they come: a workgroup
// for each row fetches the statistics side by side and then streams the partial rows
// sixteen at a time.
#include "attn_partial.h"
#include "pkv_kernels.h"

namespace pkv {
namespace {

constexpr int kBatch = 8;      // records in flight per thread
constexpr int kRowBatch = 16;  // partial rows in flight per wavefront, by rows

// kPer = D / 64 consecutive floats of a row per lane
template <int kPer> struct Chunk { typedef float T __attribute__((ext_vector_type(kPer))); };
template <> struct Chunk<1> { typedef float T; };
template <int kPer> __device__ __forceinline__ float chunk_get(const typename Chunk<kPer>::T& v, int i) { return v[i]; }
template <> __device__ __forceinline__ float chunk_get<1>(const float& v, int) { return v; }

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
// request, a segment that one wavefront finished, a batch that was cut along its segments (cumB[0] < 0).
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
// acc this lane's kPer floats of the sum of their rows weighted by 2^(m - M), and
// lsum the wave-wide sum of their partial sums with the same weights.  count = 0
// leaves (M, lsum, acc) = (-inf, 0, 0).
template <int kD>
__device__ __forceinline__ void fold_records(const AttnLaunch& a, const RowRecords& r, int begin,
                                             int stride, int count, int lane, float& M, float& lsum,
                                             float (&acc)[kD / 64]) {
  constexpr int kPer = kD / 64;
  typedef typename Chunk<kPer>::T Vec;
  const int rec_floats = record_floats(a.G, kD);
  auto record = [&](int i) -> const float* {
    return a.ws_rec + (int64_t)(r.first + begin + i * stride) * rec_floats;
  };
  auto stats = [&](int i) -> float2 {   // (max, sum) of record i for this head
    return *(const float2*)(record(i) + a.G * kD + 2 * r.g);
  };
  // the statistics of the first 64 records stay in registers for the second pass
  const float2 ml0 = (lane < count) ? stats(lane) : float2{kNegInf, 0.f};
  M = ml0.x;
  for (int i0 = 64; i0 < count; i0 += 64) {
    const int i = i0 + lane;
    if (i < count) M = fmaxf(M, stats(i).x);
  }
  M = wave_max(M);

  lsum = 0.f;
#pragma unroll
  for (int i = 0; i < kPer; ++i) acc[i] = 0.f;
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
      Vec v[kRowBatch];
      float wj[kRowBatch];
#pragma unroll
      for (int u = 0; u < kRowBatch; ++u) {
        const int j = min(j0 + u, cnt - 1);   // clamped rows get weight 0
        wj[u] = (j0 + u < cnt) ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), j)) : 0.f;
        v[u] = *((const Vec*)(record(i0 + j) + r.g * kD) + lane);
      }
#pragma unroll
      for (int u = 0; u < kRowBatch; ++u) {
        // a weight of exactly zero must also silence whatever the row holds
#pragma unroll
        for (int i = 0; i < kPer; ++i)
          acc[i] = (wj[u] != 0.f) ? __builtin_fmaf(wj[u], chunk_get<kPer>(v[u], i), acc[i]) : acc[i];
      }
    }
  }
  lsum = wave_sum(lsum);
}

// Normalise, scale, round once to bf16 and store this lane's kPer elements of the row.
template <int kPer>
__device__ __forceinline__ void store_row(uint16_t* dst, const float (&acc)[kPer], float lsum, float out_scale) {
  const float inv = lsum > 0.f ? out_scale / lsum : 0.f;
  uint16_t r[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) r[i] = (uint16_t)pack_bf16(acc[i] * inv, 0.f);
  if (kPer == 1) dst[0] = r[0];
  else if (kPer == 2) *(uint32_t*)dst = r[0] | ((uint32_t)r[1] << 16);
  else *(uint2*)dst = make_uint2(r[0] | ((uint32_t)r[1] << 16), r[2] | ((uint32_t)r[3] << 16));
}

// A row of a batch that goes by rows.  Wavefront i of the workgroup folds records i, i + n, i + 2n, ...
// (n = wavefronts in the workgroup), the partial results meet in LDS and wavefront 0 folds those.
template <int kD, int kThreads>
__device__ __forceinline__ void reduce_row(const AttnLaunch& a, int row) {
  constexpr int kPer = kD / 64, kWidth = kThreads / 64;
  __shared__ float part_stats[kWidth][2];
  __shared__ float part_acc[kWidth][kD];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  RowRecords r;
  if (!locate_records(a, row, r)) return;   // the same for every wavefront of the workgroup
  float M, lsum, acc[kPer];
  const int count = r.np > wave ? (r.np - wave + kWidth - 1) / kWidth : 0;
  fold_records<kD>(a, r, wave, kWidth, count, lane, M, lsum, acc);
  if (lane == 0) { part_stats[wave][0] = M; part_stats[wave][1] = lsum; }
#pragma unroll
  for (int i = 0; i < kPer; ++i) part_acc[wave][kPer * lane + i] = acc[i];
  __syncthreads();
  if (wave == 0) {
    float Mall = kNegInf;
    for (int w = 0; w < kWidth; ++w) Mall = fmaxf(Mall, part_stats[w][0]);
    float lall = 0.f, total[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) total[i] = 0.f;
    for (int w = 0; w < kWidth; ++w) {
      const float m = part_stats[w][0];
      if (m == kNegInf) continue;   // nothing valid behind this partial result: weight 0
      const float f = __builtin_amdgcn_exp2f(m - Mall);
      lall = __builtin_fmaf(f, part_stats[w][1], lall);
#pragma unroll
      for (int i = 0; i < kPer; ++i) total[i] = __builtin_fmaf(f, part_acc[w][kPer * lane + i], total[i]);
    }
    store_row<kPer>(a.layer.out + (int64_t)row * kD + kPer * lane, total, lall, a.out_scale);
  }
  __syncthreads();   // the next row uses the same LDS
}
template <int kD, int kThreads>
__device__ __forceinline__ void reduce_rows(const AttnLaunch& a) {
  for (int row = blockIdx.x; row < a.S * a.Hq; row += gridDim.x) reduce_row<kD, kThreads>(a, row);
}

// The segment that begins in a workgroup of the stream pass and goes on in others.  A thread owns 16 bytes
// of the rows and every sets-th record; the sets meet in LDS.
constexpr int kGroupThreads = 512;
template <int kD, typename Layers>
__device__ __forceinline__ void reduce_segment(const AttnLaunch& a, const Layers& layers, const SharedSegment& seg, int group) {
  __shared__ f32x4 rows[kGroupThreads];
  __shared__ f32x2 stats[kGroupThreads];
  const int items = a.G * (kD / 4);
  const int sets = min(max(kGroupThreads / items, 1), seg.count);
  uint16_t* out = layer_of(a, layers).out + (int64_t)seg.row * kD;
  for (int t = threadIdx.x; t < max(items, kGroupThreads); t += kGroupThreads) {
    const int set = t / items, item = t - set * items, head = item / (kD / 4);
    Partial p = kNothing;
    for (int i0 = set; set < sets && i0 < seg.count; i0 += kBatch * sets) {
      f32x4 x[kBatch];
      f32x2 ml[kBatch];
#pragma unroll
      for (int z = 0; z < kBatch; ++z) {
        const int i = min(i0 + z * sets, seg.count - 1);
        const float* rec = group_record(a, kD, layer_index(layers), group + i, i == 0);
        x[z] = *(const f32x4*)(rec + 4 * item);
        ml[z] = *(const f32x2*)(rec + a.G * kD + 2 * head);
        if (i0 + z * sets >= seg.count) ml[z].x = kNegInf;
      }
      fold(p, ml, x);
    }
    if (sets > 1) {   // then every thread is in its only turn of this loop
      rows[t] = p.x;
      stats[t] = f32x2{p.m, p.l};
      __syncthreads();
      if (set != 0) return;
      for (int z = 1; z < sets; ++z) {
        const f32x2 ml[1] = {stats[t + z * items]};
        const f32x4 x[1] = {rows[t + z * items]};
        fold(p, ml, x);
      }
    }
    if (set == 0) *(u32x2*)(out + 4 * item) = finish_row4(p.x, inverse(p.l, a.out_scale));
  }
}

// Many segments.
template <int kD, typename Layers>
__global__ __launch_bounds__(kGroupThreads) void attn_reduce_group_kernel(AttnLaunch a, Layers layers) {
  const SharedSegment seg = *shared_segment(a, layer_index(layers), blockIdx.x);
  if (seg.count > 0) reduce_segment<kD>(a, layers, seg, blockIdx.x);
}
// Few segments: whichever of the two the stream pass has chosen.  Registers as for the two wavefronts per
// SIMD that there are: left to itself the compiler has fewer loads in flight (8 requests of 6000..12000
// tokens on 8/1 heads 22.5 -> 21.7 us).
template <int kD>
__global__ __launch_bounds__(kGroupThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_reduce_few_kernel(AttnLaunch a) {
  const SharedSegment seg = *shared_segment(a, 0, blockIdx.x);
  if (seg.count == kByRows) reduce_rows<kD, kGroupThreads>(a);
  else if (seg.count > 0) reduce_segment<kD>(a, OneLayer{}, seg, blockIdx.x);
}
template <int kD, int kThreads>
__global__ __launch_bounds__(kThreads) void attn_reduce_rows_kernel(AttnLaunch a) {
  reduce_rows<kD, kThreads>(a);
}

}  // namespace

template <int kD>
static void launch_dim(const AttnLaunch& a, const AttnLayers* layers, hipStream_t stream) {
  const dim3 groups(a.waves / group_waves(kD), layers ? layers->count : 1), block(kGroupThreads);
  if (a.leaves == kManySegments) {
    if (layers) hipLaunchKernelGGL((attn_reduce_group_kernel<kD, AttnLayers>), groups, block, 0, stream, a, *layers);
    else hipLaunchKernelGGL((attn_reduce_group_kernel<kD, OneLayer>), groups, block, 0, stream, a, OneLayer{});
  } else if (a.leaves == kFewSegments) {
    hipLaunchKernelGGL(attn_reduce_few_kernel<kD>, groups, block, 0, stream, a);
  } else if (a.waves / (a.S * a.Hkv) >= 128) {
    // hundreds of records for a row: 16 wavefronts for it instead of 8 (one request of 6000..12000 tokens on
    // 8/1 heads 21.0 -> 19.2 us; 16 of 750..1500, 65 records, lose 0.9 by it)
    hipLaunchKernelGGL((attn_reduce_rows_kernel<kD, 1024>), dim3(a.S * a.Hq), dim3(1024), 0, stream, a);
  } else {
    hipLaunchKernelGGL((attn_reduce_rows_kernel<kD, 512>), dim3(a.S * a.Hq), dim3(512), 0, stream, a);
  }
}

hipError_t launch_attn_reduce(const AttnLaunch& a, const AttnLayers* layers, hipStream_t stream) {
  if (layers && a.leaves != kManySegments) return hipErrorInvalidValue;   // one layer has the whole workspace
  if (a.D == 64) launch_dim<64>(a, layers, stream);
  else if (a.D == 128) launch_dim<128>(a, layers, stream);
  else if (a.D == 256) launch_dim<256>(a, layers, stream);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace pkv
