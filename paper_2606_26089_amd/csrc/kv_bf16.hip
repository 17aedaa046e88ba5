// Truth encoder and cross K/V cache of every block in one BF16 kernel (d = 256, 8 heads of 32):
//   c = LN_t(u W_tin + b_tin) in BF16;  [K_l | V_l] = c [W_kc | W_vc]_l + b, l < L,
// written to the head-major planes [L][K, V][8 heads][cap rows][32] the attention kernel reads.
//
// A workgroup of eight waves takes 64 particles and a range of the 16 L column blocks of 32 (a
// column block is a plane): the encoding goes from the nine features through registers into an
// LDS tile of MFMA A operands, and every wave streams the weight fragments of its column blocks
// (w, w + 8, ...) from L2, eight in flight. Before, the encoding was written and read by a GEMM per
// block whose row-major result a third kernel copied into the planes: five passes over the
// activations where this one writes the cache once. Bound: those writes (6 KB a particle) and the
// products, 1.8 ms each for 1.35 M particles at the card's copy and matrix rates: 9.9 -> 3.0 ms
// (2.8 TB/s). Transposed products, whose stores are 8 bytes of a row, took 3.9 ms (9.7 with
// non-temporal stores): a row has to be written by one instruction.
// The encoding is formed in the order of k_truth_encode and the products in that of the GEMM
// (16 k at a time, the bias last), so the cache is bitwise the same.
#include "block_common.h"

namespace fmd {
namespace {

constexpr int kRingKv = 8;

// Sum over the wave in the order of wave_sum (lane bits 5 to 0): after the steps for bits 5 to b + 1
// the lanes that differ only in those hold the same value, so a rotation inside the 16-lane row
// serves as the exchange over bit b.
template <int CTRL>
__device__ __forceinline__ float plus_dpp(float v) {
  return v + __builtin_amdgcn_update_dpp(0.f, v, CTRL, 0xF, 0xF, false);
}
__device__ __forceinline__ float wave_total(float v) {
#pragma clang fp contract(off)
  const auto r32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r32[0]) + __uint_as_float(r32[1]);
  const auto r16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r16[0]) + __uint_as_float(r16[1]);
  v = plus_dpp<0x128>(v);   // row_ror 8, 4, 2, 1
  v = plus_dpp<0x124>(v);
  v = plus_dpp<0x122>(v);
  return plus_dpp<0x121>(v);
}

}  // namespace

__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_truth_kv(
    const float* __restrict__ u, int64_t n, const float* __restrict__ W_tin,
    const float* __restrict__ b_tin, const float* __restrict__ g, const float* __restrict__ s,
    const u32x4* __restrict__ Wf, const float* __restrict__ bias, bf16* __restrict__ kv,
    int64_t plane, int64_t row0, int n_blocks, int per) {
  constexpr int ROWS = 64, TM = 2, F = 9;
  __shared__ __attribute__((aligned(16))) bf16 A[ROWS * kLdA];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t m0 = (int64_t)blockIdx.x * ROWS;
  const int cb0 = blockIdx.y * per, cb1 = min(cb0 + per, n_blocks);
  u32x4 ring[kRingKv];
  auto frag = [&](int cb, int ks) { return Wf + ((int64_t)cb * kKs + ks) * 64; };
  if (cb0 + w < cb1) {
#pragma unroll
    for (int j = 0; j < kRingKv; ++j) ring[j] = frag(cb0 + w, j)[lane];
  }
  {
    // one wave per particle, eight of them: lane l owns columns l + 64 j
    float wt[4][F], bt[4], gt[4], st[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = lane + 64 * j;
      bt[j] = b_tin[c];
      gt[j] = g[c];
      st[j] = s[c];
#pragma unroll
      for (int k = 0; k < F; ++k) wt[j][k] = W_tin[k * kD + c];
    }
#pragma unroll 2
    for (int i = 0; i < ROWS / kWaves; ++i) {
      const int row = w * (ROWS / kWaves) + i;
      const float* ur = u + min(m0 + row, n - 1) * F;   // rows past the end repeat the last one
      float y[4], sum = 0.f, q = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float a = bt[j];
#pragma unroll
        for (int k = 0; k < F; ++k) a = fmaf(ur[k], wt[j][k], a);
        y[j] = a;
        sum += a;
      }
      const float mean = wave_total(sum) / kD;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float dv = y[j] - mean;
        q = fmaf(dv, dv, q);
      }
      const float rstd = rsqrtf(wave_total(q) / kD + kLnEps);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        A[row * kLdA + lane + 64 * j] = (bf16)((y[j] - mean) * rstd * gt[j] + st[j]);
    }
  }
  __syncthreads();
  const bf16* arow = A + (lane & 31) * kLdA + (lane >> 5) * 8;
  for (int cb = cb0 + w; cb < cb1; cb += kWaves) {
    asm volatile("" ::: "memory");   // the tile's reads stay in their column block
    const int nx = cb + kWaves < cb1 ? cb + kWaves : cb;
    const float bv = bias[cb * 32 + (lane & 31)];
    f32x16 acc[TM];
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < kKs; ++ks) {
      bf16x8 a[TM];
#pragma unroll
      for (int mi = 0; mi < TM; ++mi) a[mi] = *(const bf16x8*)(arow + mi * 32 * kLdA + ks * 16);
      const bf16x8 b = as_bf16x8(ring[ks % kRingKv]);
      ring[ks % kRingKv] = (ks + kRingKv < kKs ? frag(cb, ks + kRingKv) : frag(nx, ks + kRingKv - kKs))[lane];
#pragma unroll
      for (int mi = 0; mi < TM; ++mi)
        acc[mi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[mi], b, acc[mi], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(kKeepLoadsAndMfma);
    }
    const RowIo<bf16, kDh> io(kv + (int64_t)cb * plane * kDh, row0 + m0, lane & 31, lane);
    if (m0 + ROWS <= n) {
#pragma unroll
      for (int mi = 0; mi < TM; ++mi)
#pragma unroll
        for (int r = 0; r < 16; ++r) __builtin_nontemporal_store((bf16)(acc[mi][r] + bv), io.at(mi, r));
    } else {
#pragma unroll
      for (int mi = 0; mi < TM; ++mi)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (m0 + acc_row(mi, r, lane) < n) *io.at(mi, r) = (bf16)(acc[mi][r] + bv);
    }
  }
}

hipError_t launch_truth_kv(hipStream_t st, const float* u, int64_t n, const float* W_tin,
                           const float* b_tin, const float* g, const float* s, const void* Wf,
                           const float* bias, int n_layers, void* kv, int64_t plane, int64_t row0) {
  if (n <= 0) return hipSuccess;
  if (n_layers <= 0 || row0 < 0 || row0 + n > plane) return hipErrorInvalidValue;
  const int64_t tiles = (n + 63) / 64;
  if (tiles > 0x7fffffff) return hipErrorInvalidValue;
  const int blocks = 16 * n_layers;
  // Column blocks per workgroup: all of them once two workgroups a CU are filled by particles; a
  // few particles spread over the blocks (in steps of the eight waves) instead, each part forming
  // the encoding again.
  int per = blocks;
  while (per > kWaves && tiles * ((blocks + per - 1) / per) < 512) per = (per / 2 + kWaves - 1) / kWaves * kWaves;
  hipLaunchKernelGGL(k_truth_kv, dim3((unsigned)tiles, (unsigned)((blocks + per - 1) / per)),
                     dim3(kThreads), 0, st, u, n, W_tin, b_tin, g, s, (const u32x4*)Wf, bias,
                     (bf16*)kv, plane, row0, blocks, per);
  return hipGetLastError();
}

}  // namespace fmd
