// Split-K merge for paged decode attention on gfx950: folds the records (reference max, partial
// sum, un-normalised row; the maxima are in log2 units) that the stream pass left of the segments
// (request, KV head) that several of its wavefronts share into the final bf16 rows.  Segments
// that one share holds are finished there.  Bound by latency: where the records are, then the
// records.  Two layouts (pkv_kernels.h):
//
// A batch of many segments leaves at most one shared segment per workgroup of the stream pass,
// whose wavefronts have met in LDS, so that a segment has a handful of records: one workgroup
// here for each there (256), which reads one word and is done when nothing begins there.
//
// A batch of few segments (by_row) spreads each over hundreds of wavefronts, and their records come as
// they are: a wavefront or a workgroup for each row fetches the statistics side by side and then
// streams the partial rows eight at a time.
#include "attn_partial.h"
#include "pkv_kernels.h"

namespace pkv {
namespace {

constexpr int kRowsPerGroup = 4;   // wavefronts per workgroup
constexpr int kBatch = 8;          // partial rows in flight per wavefront
constexpr int kMaxWideWaves = 16;  // wavefronts of a workgroup that share one row (small batches)

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
// request, a segment that one wavefront finished, a batch that was cut along its segments.
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
    for (int j0 = 0; j0 < cnt; j0 += kBatch) {
      Vec v[kBatch];
      float wj[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int j = min(j0 + u, cnt - 1);   // clamped rows get weight 0
        wj[u] = (j0 + u < cnt) ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), j)) : 0.f;
        v[u] = *((const Vec*)(record(i0 + j) + r.g * kD) + lane);
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
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

// One wavefront per row.
template <int kD>
__global__ __launch_bounds__(kRowsPerGroup * 64) void attn_reduce_row_kernel(AttnLaunch a) {
  constexpr int kPer = kD / 64;
  const int row = blockIdx.x * kRowsPerGroup + (threadIdx.x >> 6);   // s*Hq + h
  if (row >= a.S * a.Hq) return;
  const int lane = threadIdx.x & 63;
  uint16_t* dst = a.layer.out + (int64_t)row * kD + kPer * lane;
  RowRecords r;
  if (!locate_records(a, row, r)) return;
  float M, lsum, acc[kPer];
  fold_records<kD>(a, r, 0, 1, r.np, lane, M, lsum, acc);
  store_row<kPer>(dst, acc, lsum, a.out_scale);
}

// One workgroup per row, for a small batch: few segments share the stream's
// wavefronts, so a row has up to hundreds of records and a single wavefront
// would read them in a long chain of rounds.  Wavefront i of the group folds
// records i, i + n, i + 2n, ... (n = wavefronts in the group), the partial
// results meet in LDS and wavefront 0 folds those.
template <int kD>
__global__ __launch_bounds__(kMaxWideWaves * 64) void attn_reduce_wide_row_kernel(AttnLaunch a) {
  constexpr int kPer = kD / 64;
  __shared__ float part_stats[kMaxWideWaves][2];
  __shared__ float part_acc[kMaxWideWaves][kD];
  const int row = blockIdx.x;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int width = blockDim.x >> 6;
  uint16_t* dst = a.layer.out + (int64_t)row * kD + kPer * lane;
  RowRecords r;
  if (!locate_records(a, row, r)) return;   // the same for every wavefront of the group
  float M, lsum, acc[kPer];
  const int count = r.np > wave ? (r.np - wave + width - 1) / width : 0;
  fold_records<kD>(a, r, wave, width, count, lane, M, lsum, acc);
  if (lane == 0) { part_stats[wave][0] = M; part_stats[wave][1] = lsum; }
#pragma unroll
  for (int i = 0; i < kPer; ++i) part_acc[wave][kPer * lane + i] = acc[i];
  __syncthreads();
  if (wave != 0) return;
  float Mall = kNegInf;
  for (int w = 0; w < width; ++w) Mall = fmaxf(Mall, part_stats[w][0]);
  float lall = 0.f, total[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) total[i] = 0.f;
  for (int w = 0; w < width; ++w) {
    const float m = part_stats[w][0];
    if (m == kNegInf) continue;   // nothing valid behind this partial result: weight 0
    const float f = __builtin_amdgcn_exp2f(m - Mall);
    lall = __builtin_fmaf(f, part_stats[w][1], lall);
#pragma unroll
    for (int i = 0; i < kPer; ++i) total[i] = __builtin_fmaf(f, part_acc[w][kPer * lane + i], total[i]);
  }
  store_row<kPer>(dst, total, lall, a.out_scale);
}

// One workgroup per workgroup of the stream pass: the segment that begins in that one and goes on in
// others.  A thread owns 16 bytes of the rows and every sets-th record; the sets meet in LDS.
constexpr int kGroupThreads = 512;
template <int kD, typename Layers>
__global__ __launch_bounds__(kGroupThreads) void attn_reduce_group_kernel(AttnLaunch a, Layers layers) {
  __shared__ f32x4 rows[kGroupThreads];
  __shared__ f32x2 stats[kGroupThreads];
  const int group = blockIdx.x;
  const SharedSegment seg = *shared_segment(a, blockIdx.y, group);
  if (seg.count == 0) return;
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
        const float* rec = group_record(a, kD, blockIdx.y, group + i, i == 0);
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

}  // namespace

template <int kD>
static void launch_group(const AttnLaunch& a, const AttnLayers* layers, hipStream_t stream) {
  const dim3 grid(a.waves / group_waves(kD), layers ? layers->count : 1), block(kGroupThreads);
  if (layers) hipLaunchKernelGGL((attn_reduce_group_kernel<kD, AttnLayers>), grid, block, 0, stream, a, *layers);
  else hipLaunchKernelGGL((attn_reduce_group_kernel<kD, OneLayer>), grid, block, 0, stream, a, OneLayer{});
}

hipError_t launch_attn_reduce(const AttnLaunch& a, const AttnLayers* layers, hipStream_t stream) {
  if (!a.by_row) {
    if (a.D == 64) launch_group<64>(a, layers, stream);
    else if (a.D == 128) launch_group<128>(a, layers, stream);
    else if (a.D == 256) launch_group<256>(a, layers, stream);
    else return hipErrorInvalidValue;
    return hipGetLastError();
  }
  if (layers) return hipErrorInvalidValue;   // by rows: one layer has the whole workspace
  const int rows = a.S * a.Hq;
  // A segment's records come from the wavefronts that streamed it: about
  // waves / (S * Hkv) of them when the batch is large enough to occupy them all.
  // From 32 records per row on, the row gets a workgroup of its own with one
  // wavefront per four records (8 or 16 wavefronts); below that the wider group
  // costs more than the rounds it saves (measured at 8 and 16 records per row).
  const int64_t segments = (int64_t)a.S * a.Hkv;
  const int64_t per_row = a.waves / segments;
  if (per_row >= 32) {
    const int width = per_row >= 64 ? 16 : 8;
    const dim3 grid((unsigned)rows), block(width * 64);
    if (a.D == 64) hipLaunchKernelGGL(attn_reduce_wide_row_kernel<64>, grid, block, 0, stream, a);
    else if (a.D == 128) hipLaunchKernelGGL(attn_reduce_wide_row_kernel<128>, grid, block, 0, stream, a);
    else if (a.D == 256) hipLaunchKernelGGL(attn_reduce_wide_row_kernel<256>, grid, block, 0, stream, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
  }
  dim3 grid((unsigned)((rows + kRowsPerGroup - 1) / kRowsPerGroup), 1, 1);
  const dim3 block(kRowsPerGroup * 64);
  if (a.D == 64) hipLaunchKernelGGL(attn_reduce_row_kernel<64>, grid, block, 0, stream, a);
  else if (a.D == 128) hipLaunchKernelGGL(attn_reduce_row_kernel<128>, grid, block, 0, stream, a);
  else if (a.D == 256) hipLaunchKernelGGL(attn_reduce_row_kernel<256>, grid, block, 0, stream, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace pkv
