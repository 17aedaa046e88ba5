// FP32 block segments of width 64 (the small network) on the BF16 matrix cores: the products of
// gemm_split.hip, chained on 32-row tiles.
//
//   k_gemm_oqc: attention rows -> W_o + residual -> LN2 -> cross query
//   k_gemm_mlp: attention rows -> W_oc + residual -> LN3 -> MLP + residual
//               [-> LN1 of the next block -> its Q, K and V]
//
// At this width a product is 24 to 96 matrix instructions of a wave and a kernel of its own is
// mostly its launch (4 us each, 17 an evaluation of two blocks). Bound: the chain of products and
// barriers of a tile (5 and 11 us a launch). 1,799 rows: 90 -> 66 us an evaluation, 7,081: 114 -> 85;
// where the rows fill the chip the hidden layer no longer goes through memory: 459,310 rows
// 2,646 -> 2,558 us. So every row count takes them. A workgroup of eight
// waves takes 32 rows; 16 lanes hold a row (four columns each) between the products, so the
// residual rows stay in registers and LayerNorm needs no pass of its own. Each wave multiplies at
// most one 32-column block per product, the narrow products dealt to different waves, so that
// every weight fragment a wave will need is in flight from the start. Every element is formed by
// the operations of the separate kernels in their order: the same bits.
#include "split_common.h"

namespace fmd {
namespace {

constexpr int kW = 64;                 // model width
constexpr int kRows = 32;
constexpr int kThreads = 512;
constexpr int kKs = kW / 16;           // K steps over the width
constexpr int kLdA = kW + 8;           // LDS pitch (bf16) of a plane row of the width,
constexpr int kLdH = 4 * kW + 8;       // of the hidden layer,
constexpr int kLdX = kW + 4;           // and (floats) of the FP32 rows

struct Frag {
  u32x4 q[3];
};

// the fragments of K steps [0, N) of the block at f (3 KB a step)
template <int N>
__device__ __forceinline__ void fetch(Frag (&r)[N], const char* f, int lane) {
#pragma unroll
  for (int ks = 0; ks < N; ++ks)
#pragma unroll
    for (int q = 0; q < 3; ++q) r[ks].q[q] = *(const u32x4*)(f + ks * 3072 + q * 1024 + lane * 16);
}

// one K step: the small terms first, hi hi apart
__device__ __forceinline__ void step(f32x16& hi, f32x16& lo, const bf16* __restrict__ a, int plane,
                                     const Frag& w) {
  bf16x8 x[3], b[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    x[q] = *(const bf16x8*)(a + q * plane);
    b[q] = __builtin_bit_cast(bf16x8, w.q[q]);
  }
  constexpr int ia[6] = {2, 0, 1, 1, 0, 0}, ib[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
  for (int t = 0; t < 6; ++t) {
    f32x16& acc = t == 5 ? hi : lo;
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[ia[t]], b[ib[t]], acc, 0, 0, 0);
  }
}

__device__ __forceinline__ int acc_row(int r, int lane) {
  return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
}

// (hi + lo) + bias of the 32 x 32 block of the rows in P and the weights w
__device__ __forceinline__ f32x16 block_product(const bf16* __restrict__ P, const Frag (&w)[kKs],
                                                float bias, int lane) {
  f32x16 hi, lo;
#pragma unroll
  for (int r = 0; r < 16; ++r) hi[r] = 0.f, lo[r] = 0.f;
  const bf16* a = P + (lane & 31) * kLdA + (lane >> 5) * 8;
#pragma unroll
  for (int ks = 0; ks < kKs; ++ks) step(hi, lo, a + ks * 16, kRows * kLdA, w[ks]);
#pragma unroll
  for (int r = 0; r < 16; ++r) hi[r] = (hi[r] + lo[r]) + bias;
  return hi;
}

__device__ __forceinline__ void to_rows(const f32x16& v, float* __restrict__ X, int col, int lane) {
#pragma unroll
  for (int r = 0; r < 16; ++r) X[acc_row(r, lane) * kLdX + col] = v[r];
}

__device__ __forceinline__ void to_planes(float4 v, bf16* __restrict__ P, int row, int c4) {
  bf16x4 pl[3];
  split4(v, pl);
#pragma unroll
  for (int q = 0; q < 3; ++q) *(bf16x4*)&P[q * kRows * kLdA + row * kLdA + c4] = pl[q];
}

__device__ __forceinline__ float4 plus(float4 a, float4 b) {
  return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}

// block `nb` of N columns, element (row, 32 nb + lane % 32), to C (pitch ldc)
__device__ __forceinline__ void store_block(const f32x16& v, float* __restrict__ C, int ldc, int nb,
                                            int64_t m0, int lane) {
  float* c = C + (m0 + 4 * (lane >> 5)) * ldc + nb * 32 + (lane & 31);
#pragma unroll
  for (int r = 0; r < 16; ++r) c[(8 * (r >> 2) + (r & 3)) * ldc] = v[r];
}

}  // namespace

__global__ __launch_bounds__(kThreads) void k_gemm_oqc(SplitBlockArgs p) {
  __shared__ __attribute__((aligned(16))) bf16 P[3 * kRows * kLdA];
  __shared__ __attribute__((aligned(16))) float X[kRows * kLdX];
  const int tid = threadIdx.x, lane = tid & 63, row = tid >> 4, c4 = 4 * (tid & 15);
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), nb = w & 1;
  const int64_t m0 = (int64_t)blockIdx.x * kRows;
  const float4 att = *(const float4*)(p.att + (m0 + row) * kW + c4);
  // waves 0 and 1 take W_o, 2 and 3 the cross query
  Frag wt[kKs];
  float bias = 0.f;
  if (w < 4) {
    fetch(wt, (const char*)(w < 2 ? p.Wf_o : p.Wf_qc) + nb * kKs * 3072, lane);
    bias = (w < 2 ? p.b_o : p.b_qc)[nb * 32 + (lane & 31)];
  }
  float4 h = *(const float4*)(p.H + (m0 + row) * kW + c4);
  const float4 g = *(const float4*)(p.g + c4), s = *(const float4*)(p.s + c4);
  to_planes(att, P, row, c4);
  __syncthreads();
  if (w < 2) to_rows(block_product(P, wt, bias, lane), X, nb * 32 + (lane & 31), lane);
  __syncthreads();
  h = plus(h, *(const float4*)&X[row * kLdX + c4]);
  *(float4*)(p.H + (m0 + row) * kW + c4) = h;
  to_planes(layer_norm4<16>(h, g, s, 1.0f / kW, true), P, row, c4);
  __syncthreads();
  if (w == 2 || w == 3) store_block(block_product(P, wt, bias, lane), p.qc, kW, nb, m0, lane);
}

template <bool QKV>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_gemm_mlp(
    SplitBlockArgs p) {
  __shared__ __attribute__((aligned(16))) bf16 P[3 * kRows * kLdA];
  __shared__ __attribute__((aligned(16))) bf16 Hd[3 * kRows * kLdH];
  __shared__ __attribute__((aligned(16))) float X[kRows * kLdX];
  const int tid = threadIdx.x, lane = tid & 63, row = tid >> 4, c4 = 4 * (tid & 15);
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), nb = w & 1, col = lane & 31;
  const int64_t m0 = (int64_t)blockIdx.x * kRows;
  const float4 att = *(const float4*)(p.att + (m0 + row) * kW + c4);
  // waves 0 and 1 take W_oc, 2 and 3 the down-projection (sixteen K steps, four in flight), every
  // wave a block of the up-projection, waves 0 to 5 one of Q, K and V
  constexpr int kDn = 4 * kW / 16;
  const char* dn = (const char*)p.Wf_dn + nb * kDn * 3072;
  Frag wt[kKs], wu[kKs], wq[kKs];
  float bias = 0.f;
  if (w < 4) {
    fetch(wt, w < 2 ? (const char*)p.Wf_o + nb * kKs * 3072 : dn, lane);
    bias = (w < 2 ? p.b_o : p.b_dn)[nb * 32 + col];
  }
  float4 h = *(const float4*)(p.H + (m0 + row) * kW + c4);
  fetch(wu, (const char*)p.Wf_up + w * kKs * 3072, lane);
  const float bu = p.b_up[w * 32 + col];
  const float4 g = *(const float4*)(p.g + c4), s = *(const float4*)(p.s + c4);
  float4 gn = g, sn = s;
  float bq = 0.f;
  if constexpr (QKV) {
    if (w < 6) {
      fetch(wq, (const char*)p.Wf_qkv + w * kKs * 3072, lane);
      bq = p.b_qkv[w * 32 + col];
    }
    gn = *(const float4*)(p.gn + c4);
    sn = *(const float4*)(p.sn + c4);
  }
  to_planes(att, P, row, c4);
  __syncthreads();
  if (w < 2) to_rows(block_product(P, wt, bias, lane), X, nb * 32 + col, lane);
  __syncthreads();
  h = plus(h, *(const float4*)&X[row * kLdX + c4]);
  to_planes(layer_norm4<16>(h, g, s, 1.0f / kW, true), P, row, c4);
  __syncthreads();
  {
    const f32x16 u = block_product(P, wu, bu, lane);
#pragma unroll
    for (int r = 0; r < 16; r += 4) {   // four rows of one column
      bf16x4 pl[3];
      split4(make_float4(gelu_f32(u[r]), gelu_f32(u[r + 1]), gelu_f32(u[r + 2]), gelu_f32(u[r + 3])), pl);
#pragma unroll
      for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          Hd[q * kRows * kLdH + acc_row(r + i, lane) * kLdH + w * 32 + col] = pl[q][i];
    }
  }
  __syncthreads();
  if (w == 2 || w == 3) {
    f32x16 hi, lo;
#pragma unroll
    for (int r = 0; r < 16; ++r) hi[r] = 0.f, lo[r] = 0.f;
    const bf16* a = Hd + (lane & 31) * kLdH + (lane >> 5) * 8;
#pragma unroll
    for (int ks = 0; ks < kDn; ++ks) {
      step(hi, lo, a + ks * 16, kRows * kLdH, wt[ks % kKs]);
      if (ks + kKs < kDn)
#pragma unroll
        for (int q = 0; q < 3; ++q)
          wt[ks % kKs].q[q] = *(const u32x4*)(dn + (ks + kKs) * 3072 + q * 1024 + lane * 16);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) hi[r] = (hi[r] + lo[r]) + bias;
    to_rows(hi, X, nb * 32 + col, lane);
  }
  __syncthreads();
  h = plus(h, *(const float4*)&X[row * kLdX + c4]);
  *(float4*)(p.H + (m0 + row) * kW + c4) = h;
  if constexpr (QKV) {
    to_planes(layer_norm4<16>(h, gn, sn, 1.0f / kW, true), P, row, c4);
    __syncthreads();
    if (w < 6) store_block(block_product(P, wq, bq, lane), p.qkv, 3 * kW, w, m0, lane);
  }
}

// ---------------------------------------------------------------------------------------

hipError_t launch_split_oqc(hipStream_t st, int64_t Mp, const SplitBlockArgs& a) {
  if (Mp < 0 || Mp % kRows || !a.att || !a.H || !a.Wf_o || !a.Wf_qc || !a.qc) return hipErrorInvalidValue;
  if (Mp == 0) return hipSuccess;
  hipLaunchKernelGGL(k_gemm_oqc, dim3((unsigned)(Mp / kRows)), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_split_mlp(hipStream_t st, int64_t Mp, const SplitBlockArgs& a) {
  if (Mp < 0 || Mp % kRows || !a.att || !a.H || !a.Wf_o || !a.Wf_up || !a.Wf_dn ||
      (a.Wf_qkv && (!a.gn || !a.sn || !a.b_qkv || !a.qkv)))
    return hipErrorInvalidValue;
  if (Mp == 0) return hipSuccess;
  auto* k = a.Wf_qkv ? k_gemm_mlp<true> : k_gemm_mlp<false>;
  hipLaunchKernelGGL(k, dim3((unsigned)(Mp / kRows)), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace fmd
