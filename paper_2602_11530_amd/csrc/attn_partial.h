// Partial attention results of one query row: what the stream pass and the reduce pass fold
// together (reference maximum in log2 units, partial sum, un-normalised row).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pkv {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr float kNegInf = -__builtin_huge_valf();

// Two fp32 -> packed bf16, round to nearest even (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  const f32x2 f = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
}
// A row's partial result while records are folded into it.
struct Partial {
  float m, l;
  f32x4 x;
};
constexpr Partial kNothing = {kNegInf, 0.f, {0.f, 0.f, 0.f, 0.f}};

// Folds kN partial results into p: one common maximum first, so that the weights do not wait for
// each other.  A side whose maximum is -inf (nothing valid seen) gets weight 0, and a weight of
// exactly zero also silences whatever its row holds.
template <int kN>
__device__ __forceinline__ void fold(Partial& p, const f32x2 (&ml)[kN], const f32x4 (&x)[kN]) {
  float M = p.m;
#pragma unroll
  for (int z = 0; z < kN; ++z) M = fmaxf(M, ml[z].x);
  const float w = (p.m == kNegInf) ? 0.f : __builtin_amdgcn_exp2f(p.m - M);
  p.m = M;
  p.l = (w != 0.f) ? w * p.l : 0.f;
#pragma unroll
  for (int e = 0; e < 4; ++e) p.x[e] = (w != 0.f) ? w * p.x[e] : 0.f;
#pragma unroll
  for (int z = 0; z < kN; ++z) {
    const float wz = (ml[z].x == kNegInf) ? 0.f : __builtin_amdgcn_exp2f(ml[z].x - M);
    p.l = (wz != 0.f) ? __builtin_fmaf(wz, ml[z].y, p.l) : p.l;
#pragma unroll
    for (int e = 0; e < 4; ++e) p.x[e] = (wz != 0.f) ? __builtin_fmaf(wz, x[z][e], p.x[e]) : p.x[e];
  }
}
// Normalise, scale and round once to bf16.
__device__ __forceinline__ u32x2 finish_row4(f32x4 x, float inv) {
  return u32x2{pack_bf16(x[0] * inv, x[1] * inv), pack_bf16(x[2] * inv, x[3] * inv)};
}
__device__ __forceinline__ float inverse(float l, float out_scale) {
  return l > 0.f ? out_scale / l : 0.f;
}

}  // namespace pkv
