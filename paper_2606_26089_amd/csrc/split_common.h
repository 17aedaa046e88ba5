// Helpers of the FP32 kernels on the BF16 matrix cores (gemm_split.hip, block_split.hip): three-way
// splits, LayerNorm of rows held four columns a lane, GELU.
#pragma once

#include "common.h"
#include "kernels.h"

namespace fmd {
namespace {

// x = hi + mid + lo for four values (uncontracted: the remainder is of the rounded x, also where x
// is formed by a product in the same kernel)
__device__ __forceinline__ void split4(float4 x, bf16x4 (&p)[3]) {
#pragma clang fp contract(off)
  const float v[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t hb = __float_as_uint(v[i]) & 0xffff0000u;
    const float r = v[i] - __uint_as_float(hb);
    const bf16 mid = (bf16)r;
    p[0][i] = __builtin_bit_cast(bf16, (uint16_t)(hb >> 16));
    p[1][i] = mid;
    p[2][i] = (bf16)(r - (float)mid);
  }
}

// Sum over groups of KL lanes (16, 32 or 64), the same in every lane of the group.
template <int CTRL>
__device__ __forceinline__ float dpp_plus(float v) {
  return v + __builtin_amdgcn_update_dpp(0.f, v, CTRL, 0xF, 0xF, false);
}
template <int KL>
__device__ __forceinline__ float group_sum(float v) {
  v = dpp_plus<0x128>(v);   // row_ror 8, 4, 2, 1
  v = dpp_plus<0x124>(v);
  v = dpp_plus<0x122>(v);
  v = dpp_plus<0x121>(v);
  if constexpr (KL >= 32) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  if constexpr (KL >= 64) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  return v;
}

// Exact GELU z Phi(z) to FP32 accuracy without branches (a library erf branches on |x|): with
// e = 2 Phi(-|z|) = 2^-Q(|z|), GELU = z/2 (z < 0 ? e : 2 - e). Q(a) = a P(a), P of degree 9
// fitted to -log2(2 Phi(-a)) on [0, 9.5] by Lawson's iteratively reweighted least squares,
// weighted by e (absolute error of e at most 5.3e-9), increasing up to a = 12, where e = 8e-39.
// Largest error against 64 bits 9.4e-8 |z| (the erf form with an exact erf: 1.02e-7 |z|). 16
// vector instructions, one of them the exponential.
__device__ __forceinline__ float gelu_f32(float z) {
  constexpr float c[10] = {1.15110445022583f,       0.4592188000679016f,     0.05244622007012367f,
                           -0.006953386589884758f,  6.749427029717481e-06f,  0.0002739334013313055f,
                           -7.332905806833878e-05f, 1.0027591997641139e-05f, -7.206676286841684e-07f,
                           2.1236523650713934e-08f};
  const float a = fminf(fabsf(z), 12.0f);
  float q = c[9];
#pragma unroll
  for (int k = 8; k >= 0; --k) q = fmaf(q, a, c[k]);
  const float e = __builtin_amdgcn_exp2f(-(q * a));
  return (0.5f * z) * (z < 0.f ? e : 2.0f - e);
}

// LayerNorm of a row over KL lanes, four columns a lane (inv = 1 / width; lanes past the row hold
// zeros and have in_row false). Multiply-adds are written out: the bits do not depend on the kernel.
template <int KL>
__device__ __forceinline__ float4 layer_norm4(float4 v, float4 g, float4 s, float inv, bool in_row) {
#pragma clang fp contract(off)
  const float mu = group_sum<KL>((v.x + v.y) + (v.z + v.w)) * inv;
  const float dx = v.x - mu, dy = v.y - mu, dz = v.z - mu, dw = v.w - mu;
  const float q = in_row ? fmaf(dw, dw, fmaf(dz, dz, fmaf(dy, dy, dx * dx))) : 0.f;
  const float rs = rsqrtf(fmaf(group_sum<KL>(q), inv, kLnEps));
  return make_float4(fmaf(dx * rs, g.x, s.x), fmaf(dy * rs, g.y, s.y), fmaf(dz * rs, g.z, s.z),
                     fmaf(dw * rs, g.w, s.w));
}

}  // namespace
}  // namespace fmd
