// Bandwidth-bound kernels of the sampling path: CSR token map, Philox noise, truth
// encoder, time and input embeddings, the fused output head + ODE update, ragged
// packing and parameter packing.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace fmd {

// ---------------------------------------------------------------------------------------
// Token -> event map of a CSR batch: the largest e with off[e] <= r (empty events skipped).
__global__ void k_token_map(const int64_t* __restrict__ off, int64_t E, int64_t T,
                            int32_t* __restrict__ tok_event) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= T) return;
  int64_t lo = 0, hi = E;  // off[lo] <= r < off[hi]
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (off[mid] <= r) lo = mid; else hi = mid;
  }
  tok_event[r] = (int32_t)lo;
}

hipError_t launch_token_map(hipStream_t st, const int64_t* off, int64_t E, int64_t T,
                            int32_t* tok_event) {
  if (T <= 0) return hipSuccess;
  const int64_t blocks = (T + 255) / 256;
  hipLaunchKernelGGL(k_token_map, dim3((unsigned)blocks), dim3(256), 0, st, off, E, T, tok_event);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC'11): two 64x64->128 multiplies per round,
// Weyl-sequence key schedule, ten rounds.
struct Philox4x64 {
  uint64_t c[4];
};

__device__ __forceinline__ Philox4x64 philox4x64_10(uint64_t c0, uint64_t c1, uint64_t c2,
                                                   uint64_t c3, uint64_t k0, uint64_t k1) {
  const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
  const uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) { k0 += W0; k1 += W1; }
    const uint64_t hi0 = __umul64hi(M0, c0), lo0 = M0 * c0;
    const uint64_t hi1 = __umul64hi(M1, c2), lo1 = M1 * c2;
    const uint64_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
  }
  Philox4x64 o;
  o.c[0] = c0; o.c[1] = c1; o.c[2] = c2; o.c[3] = c3;
  return o;
}

// u = ((w >> 41) + 1/2) 2^-23: exact in FP32, strictly inside (0, 1).
__device__ __forceinline__ float u23(uint64_t w) {
  return ((float)(uint32_t)(w >> 41) + 0.5f) * 1.1920928955078125e-07f;
}

__global__ void k_noise(uint64_t seed, const int64_t* __restrict__ off,
                        const int32_t* __restrict__ tok_event, int64_t T, int n_feat,
                        float* __restrict__ x, float* __restrict__ xs, int ldx) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= T) return;
  const int32_t e = tok_event[r];
  const uint64_t slot = (uint64_t)(r - off[e]);
  float z[12];
  const int nb = (n_feat + 3) >> 2;
  for (int b = 0; b < 3; ++b) {
    if (b >= nb) break;
    const Philox4x64 w = philox4x64_10((uint64_t)b, slot, (uint64_t)e, 0ull, seed, 0ull);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const float ua = u23(w.c[2 * p]), ub = u23(w.c[2 * p + 1]);
      const float rad = sqrtf(-2.0f * logf(ua));
      float sn, cs;
      sincospif(2.0f * ub, &sn, &cs);
      z[4 * b + 2 * p] = rad * cs;
      z[4 * b + 2 * p + 1] = rad * sn;
    }
  }
  float* xr = x + r * ldx;
  for (int f = 0; f < ldx; ++f) xr[f] = f < n_feat ? z[f] : 0.0f;
  if (xs) {
    float* sr = xs + r * ldx;
    for (int f = 0; f < ldx; ++f) sr[f] = f < n_feat ? z[f] : 0.0f;
  }
}

hipError_t launch_noise(hipStream_t st, uint64_t seed, const int64_t* off,
                        const int32_t* tok_event, int64_t T, int n_feat, float* x, float* xs,
                        int ldx) {
  if (T <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_noise, dim3((unsigned)((T + 255) / 256)), dim3(256), 0, st, seed, off,
                     tok_event, T, n_feat, x, xs, ldx);
  return hipGetLastError();
}

__global__ void k_philox(uint64_t k0, uint64_t k1, const uint64_t* __restrict__ ctr, int64_t n,
                         uint64_t* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint64_t* c = ctr + 4 * i;
  const Philox4x64 w = philox4x64_10(c[0], c[1], c[2], c[3], k0, k1);
  for (int k = 0; k < 4; ++k) out[4 * i + k] = w.c[k];
}

hipError_t launch_philox(hipStream_t st, uint64_t k0, uint64_t k1, const uint64_t* ctr,
                         int64_t n, uint64_t* out) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_philox, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, k0, k1, ctr, n,
                     out);
  return hipGetLastError();
}

__global__ void k_load_state(const float* __restrict__ src, int f, int64_t T,
                             float* __restrict__ x, float* __restrict__ xs, int ldx) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= T * ldx) return;
  const int64_t r = i / ldx;
  const int c = (int)(i % ldx);
  const float v = c < f ? src[r * f + c] : 0.0f;
  x[i] = v;
  if (xs) xs[i] = v;
}

hipError_t launch_load_state(hipStream_t st, const float* src, int f, int64_t T, float* x,
                             float* xs, int ldx) {
  if (T <= 0) return hipSuccess;
  const int64_t n = T * ldx;
  hipLaunchKernelGGL(k_load_state, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, src, f,
                     T, x, xs, ldx);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Truth encoder c = LN_t(u W_tin + b_tin): one wave per particle; lane owns columns
// lane + 64 j. Statistics are two-pass in registers.
constexpr int kMaxDPerLane = 16;   // d_model <= 1024

template <typename T>
__global__ __launch_bounds__(256) void k_truth_encode(
    const float* __restrict__ u, int ldu, int f, int64_t T_, const float* __restrict__ W,
    const float* __restrict__ b, const float* __restrict__ g, const float* __restrict__ s,
    int d, T* __restrict__ c, int ldc) {
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= T_) return;
  float uf[16];
  for (int k = 0; k < f; ++k) uf[k] = u[r * ldu + k];
  const int nj = d >> 6;
  float y[kMaxDPerLane];
  float sum = 0.f;
#pragma unroll
  for (int jj = 0; jj < kMaxDPerLane; ++jj) {
    if (jj < nj) {
      const int j = lane + 64 * jj;
      float a = b[j];
      for (int k = 0; k < f; ++k) a = fmaf(uf[k], W[k * d + j], a);
      y[jj] = a;
      sum += a;
    }
  }
  const float mean = wave_sum(sum) / d;
  float q = 0.f;
#pragma unroll
  for (int jj = 0; jj < kMaxDPerLane; ++jj)
    if (jj < nj) { const float dv = y[jj] - mean; q = fmaf(dv, dv, q); }
  const float rstd = rsqrtf(wave_sum(q) / d + kLnEps);
#pragma unroll
  for (int jj = 0; jj < kMaxDPerLane; ++jj)
    if (jj < nj) {
      const int j = lane + 64 * jj;
      c[r * ldc + j] = from_f32<T>((y[jj] - mean) * rstd * g[j] + s[j]);
    }
}

template <typename T>
hipError_t launch_truth_encode(hipStream_t st, const float* u, int ldu, int f, int64_t T_,
                               const float* W, const float* b, const float* g,
                               const float* s, int d, T* c, int ldc) {
  if (T_ <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_truth_encode<T>, dim3((unsigned)((T_ + 3) / 4)), dim3(256), 0, st, u,
                     ldu, f, T_, W, b, g, s, d, c, ldc);
  return hipGetLastError();
}
template hipError_t launch_truth_encode<float>(hipStream_t, const float*, int, int, int64_t,
                                               const float*, const float*, const float*,
                                               const float*, int, float*, int);
template hipError_t launch_truth_encode<bf16>(hipStream_t, const float*, int, int, int64_t,
                                              const float*, const float*, const float*,
                                              const float*, int, bf16*, int);

// ---------------------------------------------------------------------------------------
// Time embedding: temb[e, j] = b_xin[j] + b_time[j] + sum_k phi_k(t_e) W_time[k, j] with
// phi = [sin(w_k t) | cos(w_k t)], w_k = 10000^(-k/(E/2)). One block per event, or per stage of a
// call (all at once, 5 us; a launch per stage took 4.7 us of every evaluation).
__global__ __launch_bounds__(256) void k_time_embed(const float* __restrict__ t_ev,
                                                    const StageDesc* __restrict__ desc,
                                                    const float* __restrict__ W,
                                                    const float* __restrict__ b_time,
                                                    const float* __restrict__ b_xin, int E_dim,
                                                    int d, float* __restrict__ temb) {
  __shared__ float phi[64];
  const int e = blockIdx.x;
  const float t = t_ev ? t_ev[e] : desc[e].t;
  const int half = E_dim >> 1;
  if (threadIdx.x < half) {
    // ln(10000) / half scales the exponent
    const float w = expf(-(float)threadIdx.x * (9.210340371976184f / (float)half));
    float sn, cs;
    sincosf(w * t, &sn, &cs);
    phi[threadIdx.x] = sn;
    phi[threadIdx.x + half] = cs;
  }
  __syncthreads();
  for (int j = threadIdx.x; j < d; j += blockDim.x) {
    float a = 0.f;
    for (int k = 0; k < E_dim; ++k) a = fmaf(phi[k], W[k * d + j], a);
    temb[(int64_t)e * d + j] = (a + b_time[j]) + b_xin[j];
  }
}

hipError_t launch_time_embed(hipStream_t st, const float* t_ev, const StageDesc* desc, int n,
                             const float* W_time, const float* b_time, const float* b_xin,
                             int E_dim, int d, float* temb) {
  if (n <= 0) return hipSuccess;
  if (!t_ev && !desc) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_time_embed, dim3(n), dim3(256), 0, st, t_ev, desc, W_time, b_time, b_xin,
                     E_dim, d, temb);
  return hipGetLastError();
}

__global__ void k_stage_begin(StageCtl* ctl, float* out) { *ctl = StageCtl{0, 0, out}; }

hipError_t launch_stage_begin(hipStream_t st, StageCtl* ctl, float* out) {
  hipLaunchKernelGGL(k_stage_begin, dim3(1), dim3(1), 0, st, ctl, out);
  return hipGetLastError();
}

// Input embedding H = xs W_xin + temb, one wave per token (lane owns columns lane + 64 j),
// with the row's LayerNorm statistics for the first block.
__global__ __launch_bounds__(256) void k_embed(const float* __restrict__ xs, int ldx, int f,
                                               int64_t T, const int32_t* __restrict__ tok_event,
                                               const float* __restrict__ temb, StageCtl* ctl,
                                               const float* __restrict__ W, int d,
                                               float* __restrict__ H, int ldh,
                                               float2* __restrict__ stats) {
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const float* te = stage_row(temb, ctl, d);
  if (r >= T) return;
  if (tok_event) te = temb + (int64_t)tok_event[r] * d;
  float xv[16];
  for (int k = 0; k < f; ++k) xv[k] = xs[r * ldx + k];
  const int nj = d >> 6;
  float y[kMaxDPerLane];
  float sum = 0.f;
#pragma unroll
  for (int jj = 0; jj < kMaxDPerLane; ++jj)
    if (jj < nj) {
      const int j = lane + 64 * jj;
      float a = te[j];
      for (int k = 0; k < f; ++k) a = fmaf(xv[k], W[k * d + j], a);
      y[jj] = a;
      sum += a;
      H[r * ldh + j] = a;
    }
  const float mean = wave_sum(sum) / d;
  float q = 0.f;
#pragma unroll
  for (int jj = 0; jj < kMaxDPerLane; ++jj)
    if (jj < nj) { const float dv = y[jj] - mean; q = fmaf(dv, dv, q); }
  const float var = wave_sum(q) / d;
  if (lane == 0) stats[r] = make_float2(mean, rsqrtf(var + kLnEps));
}

// The same for d = 256 and 9 input features, built for memory-level parallelism: a wave
// embeds kEmbTok consecutive tokens, lane l owning columns 4l .. 4l + 3 (16-byte loads and
// stores), with W_xin kept in registers across the tokens and the token inputs read by
// scalar loads. Each output is formed in the same order as above (temb first, then the
// features in order), so H is identical; the statistics reductions of all tokens of the
// wave run side by side.
constexpr int kEmbTok = 8;
constexpr int kEmbF = 9;
__global__ __launch_bounds__(256) void k_embed256(const float* __restrict__ xs, int ldx,
                                                  int64_t T, const int32_t* __restrict__ tok_event,
                                                  const float* __restrict__ temb, StageCtl* ctl,
                                                  const float* __restrict__ W,
                                                  float* __restrict__ H, int ldh,
                                                  float2* __restrict__ stats) {
  constexpr int D = 256;
  const int lane = threadIdx.x & 63;
  const int64_t r0 =
      ((int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * kEmbTok;
  const float* stage = stage_row(temb, ctl, D);
  if (r0 >= T) return;
  float4 w[kEmbF];
#pragma unroll
  for (int k = 0; k < kEmbF; ++k) w[k] = *(const float4*)(W + k * D + 4 * lane);
  float4 a[kEmbTok];
  float part[kEmbTok];
#pragma unroll
  for (int t = 0; t < kEmbTok; ++t) {
    const int64_t r = r0 + t;
    a[t] = make_float4(0.f, 0.f, 0.f, 0.f);
    part[t] = 0.f;
    if (r < T) {
      const float* te = tok_event ? temb + (int64_t)tok_event[r] * D : stage;
      float4 v = *(const float4*)(te + 4 * lane);
#pragma unroll
      for (int k = 0; k < kEmbF; ++k) {
        const float x = xs[r * ldx + k];
        v.x = fmaf(x, w[k].x, v.x);
        v.y = fmaf(x, w[k].y, v.y);
        v.z = fmaf(x, w[k].z, v.z);
        v.w = fmaf(x, w[k].w, v.w);
      }
      *(float4*)(H + r * ldh + 4 * lane) = v;
      a[t] = v;
      part[t] = (v.x + v.y) + (v.z + v.w);
    }
  }
  float mean[kEmbTok];
#pragma unroll
  for (int t = 0; t < kEmbTok; ++t) mean[t] = wave_sum(part[t]) * (1.0f / D);
#pragma unroll
  for (int t = 0; t < kEmbTok; ++t) {
    const float dx = a[t].x - mean[t], dy = a[t].y - mean[t], dz = a[t].z - mean[t],
                dw = a[t].w - mean[t];
    part[t] = fmaf(dw, dw, fmaf(dz, dz, fmaf(dy, dy, dx * dx)));
  }
#pragma unroll
  for (int t = 0; t < kEmbTok; ++t) {
    const float var = wave_sum(part[t]) * (1.0f / D);
    if (lane == 0 && r0 + t < T) stats[r0 + t] = make_float2(mean[t], rsqrtf(var + kLnEps));
  }
}

hipError_t launch_embed(hipStream_t st, const float* xs, int ldx, int f, int64_t T,
                        const int32_t* tok_event, const float* temb, StageCtl* ctl,
                        const float* W_xin, int d, float* H, int ldh, float2* stats) {
  if (T <= 0) return hipSuccess;
  if (d == 256 && f == kEmbF && ldh % 4 == 0) {
    const int64_t waves = (T + kEmbTok - 1) / kEmbTok;
    hipLaunchKernelGGL(k_embed256, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, st, xs, ldx,
                       T, tok_event, temb, ctl, W_xin, H, ldh, stats);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_embed, dim3((unsigned)((T + 3) / 4)), dim3(256), 0, st, xs, ldx, f, T,
                     tok_event, temb, ctl, W_xin, d, H, ldh, stats);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// The linear field's whole stage. Every thread reads the stage; the thread that moves on to the
// next one does so in a launch of its own (k_linear_advance), after all have read it.
__global__ void k_linear_update(float alpha, float beta, const StageDesc* __restrict__ desc,
                                const StageCtl* __restrict__ ctl, int64_t T, int f,
                                float* __restrict__ x, float* __restrict__ acc,
                                float* __restrict__ xs, int ldx, int ldo) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= T * f) return;
  const StageDesc sd = desc[ctl->first];
  float* out = sd.write_out ? ctl->out : nullptr;
  const int64_t r = i / f;
  const int k = (int)(i % f);
  const int64_t o = r * ldx + k;
  const float v = (alpha + beta * sd.t) * xs[o];
  ode_update(sd.mode, sd.h, v, x + o, acc + o, xs + o, out ? out + r * ldo + k : nullptr);
}
__global__ void k_linear_advance(StageCtl* ctl) { ctl->first += 1; }

hipError_t launch_linear_update(hipStream_t st, float alpha, float beta, const StageDesc* desc,
                                StageCtl* ctl, int64_t T, int f, float* x, float* acc,
                                float* xs, int ldx, int ldo) {
  if (T <= 0) return hipSuccess;
  const int64_t n = T * f;
  hipLaunchKernelGGL(k_linear_update, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, alpha,
                     beta, desc, ctl, T, f, x, acc, xs, ldx, ldo);
  hipLaunchKernelGGL(k_linear_advance, dim3(1), dim3(1), 0, st, ctl);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Parameter packing and conversions.
template <typename T>
__global__ void k_pack_weight(const float* __restrict__ W, int K, int N, T* __restrict__ Wt) {
  __shared__ float tile[32][33];
  const int k0 = blockIdx.y * 32, n0 = blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 256 threads: 32 x 8
  for (int i = ty; i < 32; i += 8) {
    const int k = k0 + i, n = n0 + tx;
    tile[i][tx] = (k < K && n < N) ? W[(int64_t)k * N + n] : 0.f;
  }
  __syncthreads();
  for (int i = ty; i < 32; i += 8) {
    const int n = n0 + i, k = k0 + tx;
    if (n < N && k < K) Wt[(int64_t)n * K + k] = from_f32<T>(tile[tx][i]);
  }
}

template <typename T>
hipError_t launch_pack_weight(hipStream_t st, const float* W, int K, int N, T* Wt) {
  dim3 grid((N + 31) / 32, (K + 31) / 32);
  hipLaunchKernelGGL(k_pack_weight<T>, grid, dim3(256), 0, st, W, K, N, Wt);
  return hipGetLastError();
}
template hipError_t launch_pack_weight<float>(hipStream_t, const float*, int, int, float*);
template hipError_t launch_pack_weight<bf16>(hipStream_t, const float*, int, int, bf16*);

template <typename T>
__global__ void k_convert(const float* __restrict__ src, int64_t n, T* __restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = from_f32<T>(src[i]);
}
template <typename T>
__global__ void k_to_f32(const T* __restrict__ src, int64_t n, float* __restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = to_f32(src[i]);
}

template <typename T>
hipError_t launch_convert(hipStream_t st, const float* src, int64_t n, T* dst) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_convert<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, src, n,
                     dst);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_to_f32(hipStream_t st, const T* src, int64_t n, float* dst) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_to_f32<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, src, n,
                     dst);
  return hipGetLastError();
}
template hipError_t launch_convert<float>(hipStream_t, const float*, int64_t, float*);
template hipError_t launch_convert<bf16>(hipStream_t, const float*, int64_t, bf16*);
template hipError_t launch_to_f32<float>(hipStream_t, const float*, int64_t, float*);
template hipError_t launch_to_f32<bf16>(hipStream_t, const bf16*, int64_t, float*);

// ---------------------------------------------------------------------------------------
// Ragged packing: padded [E, n_max, f] + lengths -> CSR offsets + rows. Lengths are
// clamped to [0, n_max], so the output never exceeds E * n_max rows.
// One block computes the exclusive prefix sum (chunks of 1024 with a running carry).
__device__ __forceinline__ int64_t clamp_len(int32_t v, int n_max) {
  return v < 0 ? 0 : (v > n_max ? n_max : v);
}

__global__ __launch_bounds__(1024) void k_scan_lengths(const int32_t* __restrict__ len,
                                                       int64_t E, int n_max,
                                                       int64_t* __restrict__ off) {
  __shared__ int64_t buf[1024];
  __shared__ int64_t carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int64_t base = 0; base < E; base += 1024) {
    const int64_t i = base + threadIdx.x;
    buf[threadIdx.x] = i < E ? clamp_len(len[i], n_max) : 0;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {          // Hillis-Steele inclusive scan
      const int64_t v = threadIdx.x >= o ? buf[threadIdx.x - o] : 0;
      __syncthreads();
      buf[threadIdx.x] += v;
      __syncthreads();
    }
    if (i < E) off[i + 1] = carry + buf[threadIdx.x];
    __syncthreads();
    if (threadIdx.x == 1023) carry += buf[1023];
    __syncthreads();
  }
  if (threadIdx.x == 0) off[0] = 0;
}

__global__ void k_scatter_rows(const float* __restrict__ padded, const int32_t* __restrict__ len,
                               const int64_t* __restrict__ off, int64_t E, int n_max, int f,
                               float* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;   // (e, slot, feature)
  const int64_t per_event = (int64_t)n_max * f;
  if (i >= E * per_event) return;
  const int64_t e = i / per_event;
  const int64_t rem = i % per_event;
  const int slot = (int)(rem / f), k = (int)(rem % f);
  if (slot < clamp_len(len[e], n_max)) out[(off[e] + slot) * f + k] = padded[i];
}

hipError_t launch_pack_padded(hipStream_t st, const float* padded, const int32_t* lengths,
                              int64_t E, int n_max, int f, int64_t* off_out, float* feat_out) {
  hipLaunchKernelGGL(k_scan_lengths, dim3(1), dim3(1024), 0, st, lengths, E, n_max, off_out);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || E == 0) return e;
  const int64_t n = E * n_max * f;
  hipLaunchKernelGGL(k_scatter_rows, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, padded,
                     lengths, off_out, E, n_max, f, feat_out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Output head for d = 256 and 9 features: v = LN_f(H) W_out + b_out followed by the ODE
// update of the state (the same update as the GEMM head's epilogue). The product has only
// nine columns, so it runs on the vector ALUs in FP32 instead of a matrix tile padded to 64
// columns: half a wave per token (lane i of the half owns columns 4i .. 4i+3 and 128 + 4i ..
// 131 + 4i, coalesced 16-byte loads), W_out, gain and shift in registers, the nine dot
// products reduced over the half wave by DPP rotations inside 16-lane rows and one
// permlane16 swap between the two rows. Lanes 0..8 of a half then update feature i.
namespace {
constexpr int kHeadIter = 4;     // token pairs per wave
constexpr int kHeadF = 9;

template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __builtin_amdgcn_update_dpp(0.f, v, CTRL, 0xF, 0xF, false);
}

// Sum over the 32 lanes of each half wave, left in every lane of the half; the same
// addition tree for both halves and for every lane.
__device__ __forceinline__ float half_wave_sum(float v) {
  v = dpp_add<0x128>(v);   // row_ror 8
  v = dpp_add<0x124>(v);   // row_ror 4
  v = dpp_add<0x122>(v);   // row_ror 2
  v = dpp_add<0x121>(v);   // row_ror 1
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                  false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
}  // namespace

__global__ __launch_bounds__(256) void k_head256(const float* __restrict__ H,
                                                 const float2* __restrict__ stats,
                                                 const float* __restrict__ g,
                                                 const float* __restrict__ s,
                                                 const float* __restrict__ Wt,
                                                 const float* __restrict__ b, OdeArgs ode) {
  constexpr int D = 256;
  const int lane = threadIdx.x & 63, half = lane >> 5, i = lane & 31;
  const int64_t p0 =
      ((int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * kHeadIter;
  const int64_t T = ode.m_valid;
  if (2 * p0 >= T) return;
  float4 hv[kHeadIter][2];
  float2 st[kHeadIter];
#pragma unroll
  for (int it = 0; it < kHeadIter; ++it) {
    const int64_t r = min(2 * (p0 + it) + half, T - 1);
#pragma unroll
    for (int j = 0; j < 2; ++j) hv[it][j] = *(const float4*)(H + r * D + 128 * j + 4 * i);
    st[it] = stats[r];
  }
  float4 gv[2], sv[2], w[kHeadF][2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    gv[j] = *(const float4*)(g + 128 * j + 4 * i);
    sv[j] = *(const float4*)(s + 128 * j + 4 * i);
#pragma unroll
    for (int c = 0; c < kHeadF; ++c) w[c][j] = *(const float4*)(Wt + c * D + 128 * j + 4 * i);
  }
  const OdeStage os = ode_stage(ode);
  float* out = os.out;
  ode_next_stage(ode);
  const float bias = i < kHeadF ? b[i] : 0.f;
#pragma unroll
  for (int it = 0; it < kHeadIter; ++it) {
    const int64_t r = 2 * (p0 + it) + half;
    float part[kHeadF];
#pragma unroll
    for (int c = 0; c < kHeadF; ++c) part[c] = 0.f;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const float y[4] = {fmaf((hv[it][j].x - st[it].x) * st[it].y, gv[j].x, sv[j].x),
                          fmaf((hv[it][j].y - st[it].x) * st[it].y, gv[j].y, sv[j].y),
                          fmaf((hv[it][j].z - st[it].x) * st[it].y, gv[j].z, sv[j].z),
                          fmaf((hv[it][j].w - st[it].x) * st[it].y, gv[j].w, sv[j].w)};
#pragma unroll
      for (int c = 0; c < kHeadF; ++c) {
        part[c] = fmaf(y[0], w[c][j].x, part[c]);
        part[c] = fmaf(y[1], w[c][j].y, part[c]);
        part[c] = fmaf(y[2], w[c][j].z, part[c]);
        part[c] = fmaf(y[3], w[c][j].w, part[c]);
      }
    }
    float v = 0.f;
#pragma unroll
    for (int c = 0; c < kHeadF; ++c) {
      const float tot = half_wave_sum(part[c]);
      v = i == c ? tot : v;
    }
    if (i < kHeadF && r < T) {
      const int64_t o = r * ode.ldx + i;
      if (ode.tok_event) {
        const StageDesc sd = ode.desc[ode.tok_event[r]];
        ode_update(sd.mode, sd.h, v + bias, ode.x + o, ode.acc + o, ode.xs + o,
                   out && sd.write_out ? out + r * ode.ldo + i : nullptr);
      } else {
        ode_update(os.mode, os.h, v + bias, ode.x + o, ode.acc + o, ode.xs + o,
                   out ? out + r * ode.ldo + i : nullptr);
      }
    }
  }
}

// The same output head for d = 32 NV (64 to 256) on the FP32 path, with the LayerNorm statistics
// formed from the rows in registers, so no kernel has to leave them: half a wave per token, lane
// i of the half owning columns 64 c + 2i and 64 c + 2i + 1. Bound: the rows' read (448,552 rows of
// 256: 236 us, against 158 with statistics given, which cost each residual product a pass of its
// own over its sums); few rows: its launch (1,799 rows of 64: 4.5 us).
template <int NV>
__global__ __launch_bounds__(256) void k_head_rows(const float* __restrict__ H,
                                                   const float* __restrict__ g,
                                                   const float* __restrict__ s,
                                                   const float* __restrict__ Wt,
                                                   const float* __restrict__ b, OdeArgs ode) {
  constexpr int D = 32 * NV, NC = NV / 2, kIter = 2;
  const int lane = threadIdx.x & 63, half = lane >> 5, i = lane & 31;
  const int64_t p0 =
      ((int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * kIter;
  const int64_t T = ode.m_valid;
  if (2 * p0 >= T) return;
  float x[kIter][NV];
#pragma unroll
  for (int it = 0; it < kIter; ++it) {
    const int64_t r = min(2 * (p0 + it) + half, T - 1);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const float2 h = *(const float2*)(H + r * D + 64 * c + 2 * i);
      x[it][2 * c] = h.x;
      x[it][2 * c + 1] = h.y;
    }
  }
  float gv[NV], sv[NV], w[kHeadF][NV];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int col = 64 * c + 2 * i + k;
      gv[2 * c + k] = g[col];
      sv[2 * c + k] = s[col];
#pragma unroll
      for (int f = 0; f < kHeadF; ++f) w[f][2 * c + k] = Wt[f * D + col];
    }
  const OdeStage os = ode_stage(ode);
  float* out = os.out;
  ode_next_stage(ode);
  const float bias = i < kHeadF ? b[i] : 0.f;
#pragma unroll
  for (int it = 0; it < kIter; ++it) {
    const int64_t r = 2 * (p0 + it) + half;
    float sum = 0.f, sq = 0.f;
#pragma unroll
    for (int k = 0; k < NV; ++k) sum += x[it][k];
    const float mu = half_wave_sum(sum) * (1.0f / D);
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      x[it][k] -= mu;
      sq = fmaf(x[it][k], x[it][k], sq);
    }
    const float rs = rsqrtf(half_wave_sum(sq) * (1.0f / D) + kLnEps);
    float part[kHeadF];
#pragma unroll
    for (int f = 0; f < kHeadF; ++f) part[f] = 0.f;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const float y = fmaf(x[it][k] * rs, gv[k], sv[k]);
#pragma unroll
      for (int f = 0; f < kHeadF; ++f) part[f] = fmaf(y, w[f][k], part[f]);
    }
    float v = 0.f;
#pragma unroll
    for (int f = 0; f < kHeadF; ++f) {
      const float tot = half_wave_sum(part[f]);
      v = i == f ? tot : v;
    }
    if (i < kHeadF && r < T) {
      const int64_t o = r * ode.ldx + i;
      if (ode.tok_event) {
        const StageDesc sd = ode.desc[ode.tok_event[r]];
        ode_update(sd.mode, sd.h, v + bias, ode.x + o, ode.acc + o, ode.xs + o,
                   out && sd.write_out ? out + r * ode.ldo + i : nullptr);
      } else {
        ode_update(os.mode, os.h, v + bias, ode.x + o, ode.acc + o, ode.xs + o,
                   out ? out + r * ode.ldo + i : nullptr);
      }
    }
  }
}

hipError_t launch_head_rows(hipStream_t st, int d, const float* H, const float* g, const float* s,
                            const float* Wt, const float* b, const OdeArgs& ode) {
  if (ode.nf != kHeadF || d % 64 || d < 64 || d > 256) return hipErrorInvalidValue;
  if (ode.m_valid <= 0) return hipSuccess;
  auto* k = d == 64 ? k_head_rows<2> : d == 128 ? k_head_rows<4> : d == 192 ? k_head_rows<6> : k_head_rows<8>;
  hipLaunchKernelGGL(k, dim3((unsigned)((ode.m_valid + 15) / 16)), dim3(256), 0, st, H, g, s, Wt, b, ode);
  return hipGetLastError();
}

bool head256_supported(int d, int nf) { return d == 256 && nf == kHeadF; }

hipError_t launch_head256(hipStream_t st, const float* H, const float2* stats, const float* g,
                          const float* s, const float* Wt, const float* b, const OdeArgs& ode) {
  if (ode.nf != kHeadF) return hipErrorInvalidValue;
  if (ode.m_valid <= 0) return hipSuccess;
  const int64_t waves = (ode.m_valid + 2 * kHeadIter - 1) / (2 * kHeadIter);
  hipLaunchKernelGGL(k_head256, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, st, H, stats, g,
                     s, Wt, b, ode);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// One block's cross K/V rows [rows][2d] (K | V, row-major, pitch 2d) into head-major planes:
// element (row, s, head, i) -> dst[((s * n_heads + head) * plane + row0 + row) * dh + i],
// s = 0 for K, 1 for V. 16-byte copies.
__global__ void k_kv_headmajor(const bf16* __restrict__ src, int64_t rows, int d, int dh,
                               int n_heads, bf16* __restrict__ dst, int64_t plane, int64_t row0) {
  const int per_row = 2 * d / 8;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= rows * per_row) return;
  const int64_t row = t / per_row;
  const int col = (int)(t % per_row) * 8;
  const int sel = col / d, head = (col % d) / dh, i = col % dh;
  *(u32x4*)(dst + ((int64_t)(sel * n_heads + head) * plane + row0 + row) * dh + i) =
      *(const u32x4*)(src + row * 2 * d + col);
}

hipError_t launch_kv_headmajor(hipStream_t st, const void* src, int64_t rows, int d, int dh,
                               int n_heads, void* dst, int64_t plane, int64_t row0) {
  if (rows <= 0) return hipSuccess;
  if (dh % 8 || d % dh || row0 + rows > plane) return hipErrorInvalidValue;
  const int64_t n = rows * (2 * d / 8);
  hipLaunchKernelGGL(k_kv_headmajor, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                     (const bf16*)src, rows, d, dh, n_heads, (bf16*)dst, plane, row0);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Event observables of reconstructed events (Sec. 2.4, event post-processing): H_T and MET
// per event, and the isolation of every electron and muon: the pT sum of the event's other
// particles inside Delta R < 0.4, over the lepton's pT. One workgroup per event. pT, the
// trigonometric terms and every sum are FP64; the class maximum and the cone test are taken
// in FP32 with separate multiplies and adds (integer decisions in the input's precision).
// Each particle is decoded once into an LDS tile (an event of up to kObsTile particles is one
// tile; longer ones stage their tiles again for every batch of leptons) while its leptons are
// gathered, so that the cone sums run on leptons only, four threads each taking every fourth
// particle: with a thread per particle two of five waves' lanes did all of that work, one
// particle at a time, and every particle was decoded three times.
namespace {
constexpr int kObsTile = 1024;
constexpr float kObsTwoPi = (float)(2.0 * 3.14159265358979323846);
constexpr float kObsInvTwoPi = (float)(1.0 / (2.0 * 3.14159265358979323846));

__device__ __forceinline__ int obs_class(const float* f) {
  int c = 0;
  float best = f[3];
#pragma unroll
  for (int k = 1; k < 5; ++k)
    if (f[3 + k] > best) best = f[3 + k], c = k;    // first maximum
  return c;
}

__device__ __forceinline__ bool obs_in_cone(float eta_i, float phi_i, float eta_j, float phi_j) {
#pragma clang fp contract(off)
  const float deta = eta_i - eta_j;
  const float d = phi_i - phi_j;
  const float dphi = d - kObsTwoPi * rintf(d * kObsInvTwoPi);
  return deta * deta + dphi * dphi < 0.16f;
}

// Sum over the wave, pairs across lane bits 5 to 0 in turn: half and row swaps, then rotations in
// the 16-lane rows (after the bits above, lanes that differ only in those hold the same value, so
// a rotation by 2^b serves as the exchange over bit b). No LDS permutes, which a workgroup of two
// waves waits for.
template <int CTRL>
__device__ __forceinline__ double obs_plus_ror(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xF, 0xF, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, false);
  return v + __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
template <typename S>
__device__ __forceinline__ double obs_plus_swap(double v, S&& swap) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const auto lo = swap((uint32_t)u), hi = swap((uint32_t)(u >> 32));
  return __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]) +
         __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
}
__device__ __forceinline__ double obs_wave_sum(double v) {
  v = obs_plus_swap(v, [](uint32_t x) { return __builtin_amdgcn_permlane32_swap(x, x, false, false); });
  v = obs_plus_swap(v, [](uint32_t x) { return __builtin_amdgcn_permlane16_swap(x, x, false, false); });
  v = obs_plus_ror<0x128>(v);   // row_ror 8, 4, 2, 1
  v = obs_plus_ror<0x124>(v);
  v = obs_plus_ror<0x122>(v);
  return obs_plus_ror<0x121>(v);
}

// A workgroup per event: a launch has at most 2^32 - 1 work items, and the runtime cuts a larger
// grid short without an error, so millions of events go in parts (of 512 threads at most each).
template <typename F>
hipError_t event_parts(int64_t n_events, F&& launch) {
  constexpr int64_t kPart = 1 << 22;
  for (int64_t e0 = 0; e0 < n_events; e0 += kPart) {
    launch(e0, (unsigned)std::min(kPart, n_events - e0));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

struct ObsItem {       // a decoded particle, 16 bytes
  double pt;
  float eta, phi;
};
constexpr int kObsParts = 4;          // threads per lepton
// Running sums of an event: particle i adds to number i % 256, in order of i, whatever the number
// of threads, so that an event's bits do not depend on the call around it.
constexpr int kObsSums = 256;
struct ObsSums {
  double h = 0.0, px = 0.0, py = 0.0;
  __device__ __forceinline__ void add(double pt, double cs, double sn) {
    h += pt;
    px = fma(pt, cs, px);
    py = fma(pt, sn, py);
  }
};
struct ObsTerm {
  double pt, cs, sn;
};
}  // namespace

template <int NT>
__global__ __launch_bounds__(NT) void k_event_observables(const float* __restrict__ feat, int ldf,
                                                          const int64_t* __restrict__ off,
                                                          float* __restrict__ ht,
                                                          float* __restrict__ met,
                                                          float* __restrict__ iso) {
  __shared__ ObsItem item[kObsTile];
  __shared__ ObsTerm upper[NT > kObsSums ? NT - kObsSums : 1];   // terms of the threads past the sums
  __shared__ uint16_t lep[kObsTile];             // the tile's leptons, in any order
  __shared__ int n_lep;
  __shared__ double red[kObsSums / 64][3];
  const int e = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t a = off[e], n = off[e + 1] - a;
  const bool one_tile = n <= kObsTile;
  auto decode = [&](const float* f) { return ObsItem{10.0 * exp((double)f[0]), f[1], f[2]}; };
  ObsSums sums;
  // the sum of running sums 64 w to 64 w + 63
  auto reduce = [&](int w) {
    const double h = obs_wave_sum(sums.h), px = obs_wave_sum(sums.px), py = obs_wave_sum(sums.py);
    if (lane == 0) red[w][0] = h, red[w][1] = px, red[w][2] = py;
  };
  if (tid < kObsSums / 64 * 3) red[tid / 3][tid % 3] = 0.0;
  for (int64_t i0 = 0; i0 < n; i0 += kObsTile) {
    const int nt = (int)min<int64_t>(kObsTile, n - i0);
    if (i0) __syncthreads();                     // the tile before is consumed
    if (tid == 0) n_lep = 0;
    __syncthreads();
    for (int c = 0; c < nt; c += NT) {
      const int i = c + tid;
      bool is_lep = false;
      if (i < nt) {
        const float* f = feat + (a + i0 + i) * ldf;
        const ObsItem it = decode(f);
        double sn, cs;
        sincos((double)it.phi, &sn, &cs);
        if (NT <= kObsSums || tid < kObsSums)
          sums.add(it.pt, cs, sn);
        else
          upper[tid - kObsSums] = ObsTerm{it.pt, cs, sn};
        item[i] = it;
        const int cl = obs_class(f);
        is_lep = cl == 1 || cl == 2;             // electron, muon
        if (!is_lep) iso[a + i0 + i] = __builtin_nanf("");
      }
      const uint64_t bal = __ballot(is_lep);
      if (bal) {
        int base = 0;
        if (lane == 0) base = atomicAdd(&n_lep, __popcll(bal));
        base = __shfl(base, 0, kWave);
        if (is_lep) lep[base + __popcll(bal & (lane ? ~0ull >> (64 - lane) : 0ull))] = (uint16_t)i;
      }
      if constexpr (NT < kObsSums) {             // (events of up to 256: one term a running sum)
        if (c + wave * 64 < nt) reduce(c / 64 + wave);
        sums = ObsSums{};
      }
      if constexpr (NT > kObsSums) {
        static_assert(NT == 2 * kObsSums, "one upper term per running sum");
        __syncthreads();
        if (tid < kObsSums && c + kObsSums + tid < nt)
          sums.add(upper[tid].pt, upper[tid].cs, upper[tid].sn);
        __syncthreads();                         // the upper terms are rewritten
      }
    }
    __syncthreads();
    const int nl = n_lep, part = tid % kObsParts;
    for (int b0 = 0; b0 < nl; b0 += NT / kObsParts) {
      const int b = b0 + tid / kObsParts;
      const bool on = b < nl;
      const int64_t i = i0 + (on ? lep[b] : 0);
      const ObsItem me = one_tile ? item[i] : decode(feat + (a + i) * ldf);
      double sum = 0.0;
      for (int64_t j0 = 0; j0 < n; j0 += kObsTile) {
        const int mt = (int)min<int64_t>(kObsTile, n - j0);
        if (!one_tile) {
          __syncthreads();
          for (int j = tid; j < mt; j += NT) item[j] = decode(feat + (a + j0 + j) * ldf);
          __syncthreads();
        }
        if (on) {
          const int self = i >= j0 && i < j0 + mt ? (int)(i - j0) : -1;
#pragma unroll 4
          for (int j = part; j < mt; j += kObsParts) {
            const ObsItem o = item[j];
            const bool in = obs_in_cone(me.eta, me.phi, o.eta, o.phi) && j != self;
            sum += in ? o.pt : 0.0;
          }
        }
      }
#pragma unroll
      for (int o = 1; o < kObsParts; o <<= 1) sum += __shfl_xor(sum, o, kWave);
      if (on && part == 0) iso[a + i] = (float)(sum / me.pt);
    }
  }
  if (NT >= kObsSums && wave * 64 < min<int64_t>(n, kObsSums)) reduce(wave);
  __syncthreads();
  if (tid == 0) {
    double t[3] = {0.0, 0.0, 0.0};
    for (int q = 0; q < kObsSums / 64; ++q)
      for (int k = 0; k < 3; ++k) t[k] += red[q][k];
    ht[e] = (float)t[0];
    met[e] = (float)sqrt(t[1] * t[1] + t[2] * t[2]);
  }
}

hipError_t launch_event_observables(hipStream_t st, const float* feat, int ldf,
                                    const int64_t* off_device, int64_t n_events, int64_t max_n,
                                    float* ht, float* met, float* iso) {
  if (n_events <= 0) return hipSuccess;
  if (n_events > 0x7fffffff || ldf < 8) return hipErrorInvalidValue;
  // Threads per event: enough events fill the chip, and idle threads of small ones then cost more
  // than they shorten (4096 events of 20-200: 61 us a call with 128, 63 with 256, 77 with 512;
  // 16,384 heavy-tailed ones of up to 1000: 237, 180 and 230); few events are bound by the
  // longest one (64 heavy-tailed: 92, 60 and 46 us; before, a thread per particle: 88, 545, 238)
  // 128 threads hold one term a running sum, so their events have at most 256 particles.
  const bool small = max_n <= kObsSums;
  const int nt = n_events > 2048 ? (small ? 128 : 256) : n_events > 512 && small ? 256 : 512;
  auto* k = nt == 128   ? k_event_observables<128>
            : nt == 256 ? k_event_observables<256>
                        : k_event_observables<512>;
  return event_parts(n_events, [&](int64_t e0, unsigned n) {
    hipLaunchKernelGGL(k, dim3(n), dim3(nt), 0, st, feat, ldf, off_device + e0, ht + e0, met + e0, iso);
  });
}

// ---------------------------------------------------------------------------------------
// Truth preprocessing before the sampler: the model's pT cut and particle limit (stream
// compaction per event). Pass 1, one workgroup per event: a particle survives when
// x0 > c0 (x0 = ln(pT / 10 GeV), c0 = ln(cut / 10 GeV) in float32); if more than `limit`
// survive, the `limit` largest x0 are kept (equal x0: the earlier particles). Writes keep[row]
// and the event's count. A prefix sum turns the counts into the output offsets, and pass 2 writes
// the kept rows in input order.
// The cut-off of an event above the limit is found by radix selection on order-preserving
// integer keys: four histograms of eight bits, linear in the event where a rank per particle was
// quadratic (64 heavy-tailed events of up to 1000: 224 -> 53 us a call; 4096 of 20-200: 48 -> 14 us
// a launch). Pass 2 copies an event as one run of floats, not a row per thread (19 -> 10 us). With
// the prefix sum on the device (4 us) the host waits once, for the offsets: 123 -> 66 us a call.
namespace {
constexpr int kSelKeys = 2048;        // keys held in LDS; longer events read theirs again

// Order-preserving key of a survivor: larger x, larger key; +0 and -0 alike; never 0.
__device__ __forceinline__ uint32_t sel_key(float x) {
  const uint32_t b = __float_as_uint(x + 0.f);
  return b ^ ((b >> 31) ? 0xffffffffu : 0x80000000u);
}
}  // namespace

__global__ __launch_bounds__(256) void k_select_count(const float* __restrict__ feat, int ldf,
                                                      const int64_t* __restrict__ off, float c0,
                                                      int limit, uint8_t* __restrict__ keep,
                                                      int32_t* __restrict__ cnt) {
  __shared__ uint32_t s_key[kSelKeys];   // 0: not a survivor
  __shared__ int s_n[4], s_hist[256], s_bin, s_above;
  const int e = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t a = off[e], n = off[e + 1] - a;
  auto load_key = [&](int64_t i) -> uint32_t {
    const float x = feat[(a + i) * ldf];
    return x > c0 ? sel_key(x) : 0u;
  };
  int mine = 0;
  for (int64_t i = tid; i < n; i += 256) {
    const uint32_t k = load_key(i);
    if (i < kSelKeys) s_key[i] = k;
    mine += k != 0;
  }
  auto key = [&](int64_t i) { return i < kSelKeys ? s_key[i] : load_key(i); };   // own particles
  for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o, kWave);
  if (lane == 0) s_n[wave] = mine;
  __syncthreads();
  const int surv = s_n[0] + s_n[1] + s_n[2] + s_n[3];
  if (tid == 0) cnt[e] = min(surv, limit);
  if (surv <= limit || limit <= 0) {
    for (int64_t i = tid; i < n; i += 256) keep[a + i] = limit > 0 && key(i) != 0;
    return;
  }
  // the limit-th largest key, eight bits at a time: `need` keys are left to take among those
  // that agree with `top` in the bits fixed so far
  uint32_t top = 0, fixed = 0;
  int need = limit;
  for (int shift = 24; shift >= 0; shift -= 8) {
    s_hist[tid] = 0;
    __syncthreads();
    for (int64_t i = tid; i < n; i += 256) {
      const uint32_t k = key(i);
      if (k != 0 && (k & fixed) == top) atomicAdd(&s_hist[(k >> shift) & 255], 1);
    }
    __syncthreads();
    if (wave == 0) {
      // lane l: bins 255 - 4l .. 252 - 4l, largest keys first; the bin where the running count
      // reaches `need`
      int c[4], sum = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) sum += c[q] = s_hist[255 - 4 * lane - q];
      int run = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(run, o, kWave);
        if (lane >= o) run += v;
      }
      int before = run - sum;
      if (before < need && run >= need) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (before < need && before + c[q] >= need) s_bin = 255 - 4 * lane - q, s_above = before;
          before += c[q];
        }
      }
    }
    __syncthreads();
    need -= s_above;
    top |= (uint32_t)s_bin << shift;
    fixed |= 255u << shift;
    __syncthreads();   // s_bin and s_hist are rewritten
  }
  // keys above `top` stay, and the first `need` of those equal to it
  int taken = 0;
  for (int64_t i0 = 0; i0 < n; i0 += 256) {
    const int64_t i = i0 + tid;
    const uint32_t k = i < n ? key(i) : 0;
    const bool eq = k == top;
    const uint64_t bal = __ballot(eq);
    if (lane == 0) s_n[wave] = __popcll(bal);
    __syncthreads();
    int before = taken + __popcll(bal & (lane ? ~0ull >> (64 - lane) : 0ull));
    for (int q = 0; q < 4; ++q) {
      if (q < wave) before += s_n[q];
      taken += s_n[q];
    }
    if (i < n) keep[a + i] = k > top || (eq && before < need);
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void k_select_write(const float* __restrict__ feat, int ldf,
                                                      const int64_t* __restrict__ off,
                                                      const int64_t* __restrict__ off_out,
                                                      const uint8_t* __restrict__ keep,
                                                      float* __restrict__ out) {
  constexpr int kRows = 256;
  __shared__ int s_tot[4];
  __shared__ int16_t s_pos[kRows];       // kept row -> position in the chunk's output, else -1
  const int e = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t a = off[e], n = off[e + 1] - a;
  int64_t base = off_out[e];
  for (int64_t i0 = 0; i0 < n; i0 += kRows) {
    const int64_t i = i0 + tid;
    const bool k = i < n && keep[a + i];
    // block prefix of the flags: ballot within the wave, wave totals through LDS
    const uint64_t bal = __ballot(k);
    if (lane == 0) s_tot[wave] = __popcll(bal);
    __syncthreads();
    int before = __popcll(bal & (lane ? ~0ull >> (64 - lane) : 0ull));
    for (int q = 0; q < wave; ++q) before += s_tot[q];
    s_pos[tid] = k ? (int16_t)before : (int16_t)-1;
    __syncthreads();
    const int floats = (int)min<int64_t>(kRows, n - i0) * ldf;
    const float* src = feat + (a + i0) * ldf;
    float* dst = out + base * ldf;
    for (int t = tid; t < floats; t += 256) {
      const int row = t / ldf, pos = s_pos[row];
      if (pos >= 0) dst[pos * ldf + (t - row * ldf)] = src[t];
    }
    base += s_tot[0] + s_tot[1] + s_tot[2] + s_tot[3];
    __syncthreads();                     // s_tot and s_pos are rewritten
  }
}

// Exclusive prefix sum of the per-event counts into int64 offsets (off[0] = 0, off[E] = total),
// one workgroup: wave w of the sixteen scans events 64 per step in registers, sixteen such runs a
// round, the running total carried through LDS.
__global__ __launch_bounds__(1024) void k_select_offsets(const int32_t* __restrict__ cnt, int64_t E,
                                                         int64_t* __restrict__ off) {
  constexpr int kPer = 4;                // events per thread and round
  __shared__ int64_t s_wave[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int64_t carry = 0;
  for (int64_t e0 = 0; e0 < E; e0 += 1024 * kPer) {
    const int64_t i0 = e0 + (int64_t)tid * kPer;
    int c[kPer], sum = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) sum += c[q] = i0 + q < E ? cnt[i0 + q] : 0;
    int64_t run = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int64_t v = __shfl_up(run, o, kWave);
      if (lane >= o) run += v;
    }
    if (lane == 63) s_wave[wave] = run;
    __syncthreads();
    int64_t p = carry + run - sum;
    for (int q = 0; q < 16; ++q) {
      if (q < wave) p += s_wave[q];
      carry += s_wave[q];
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q)
      if (i0 + q < E) off[i0 + q] = p, p += c[q];
    __syncthreads();                     // s_wave is rewritten
  }
  if (tid == 0) off[E] = carry;
}

// Reco multiplicity per event (a stand-in law; the model can emit particles that match no
// truth particle, Sec. 2.2): N_reco = min(n_max, N - lost + fakes) for N > 0 truth particles,
// else 0. lost counts the words w_i, i < N, below thr_q (each truth particle missed with
// probability q), fakes the words w_(N + j), j < M, below thr_p (M trials of probability p).
// The words are those of Philox4x64-10 with key (seed, 1) at counters (c, e, 0, 0), four per
// counter in order. One wave per event: lane l takes counters l, l + 64, ...; the integer
// counts are summed across the wave (order-free).
__global__ __launch_bounds__(64) void k_reco_counts(const int64_t* __restrict__ off, int64_t E,
                                                    uint64_t seed, uint64_t thr_q, uint64_t thr_p,
                                                    int M, int n_max, int32_t* __restrict__ cnt) {
  const int64_t e = blockIdx.x;
  if (e >= E) return;
  const int lane = threadIdx.x;
  const int64_t n = off[e + 1] - off[e];
  if (n <= 0) {
    if (lane == 0) cnt[e] = 0;
    return;
  }
  const int64_t words = n + M, ctrs = (words + 3) / 4;
  int lost = 0, fakes = 0;
  for (int64_t c = lane; c < ctrs; c += 64) {
    const Philox4x64 w = philox4x64_10((uint64_t)c, (uint64_t)e, 0ull, 0ull, seed, 1ull);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t i = 4 * c + k;
      if (i < n) lost += w.c[k] < thr_q;
      else if (i < words) fakes += w.c[k] < thr_p;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lost += __shfl_xor(lost, o, 64);
    fakes += __shfl_xor(fakes, o, 64);
  }
  if (lane == 0) cnt[e] = (int32_t)min<int64_t>(n_max, n - lost + fakes);
}

hipError_t launch_reco_counts(hipStream_t st, const int64_t* off, int64_t n_events, uint64_t seed,
                              uint64_t thr_q, uint64_t thr_p, int fake_trials, int n_max,
                              int32_t* cnt) {
  if (n_events <= 0) return hipSuccess;
  if (n_events > 0x7fffffff || fake_trials < 0 || n_max < 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_reco_counts, dim3((unsigned)n_events), dim3(64), 0, st, off, n_events, seed,
                     thr_q, thr_p, fake_trials, n_max, cnt);
  return hipGetLastError();
}

hipError_t launch_select_count(hipStream_t st, const float* feat, int ldf, const int64_t* off,
                               int64_t n_events, float c0, int limit, uint8_t* keep,
                               int32_t* cnt) {
  if (n_events <= 0) return hipSuccess;
  if (n_events > 0x7fffffff || limit < 0) return hipErrorInvalidValue;
  return event_parts(n_events, [&](int64_t e0, unsigned n) {
    hipLaunchKernelGGL(k_select_count, dim3(n), dim3(256), 0, st, feat, ldf, off + e0, c0, limit, keep,
                       cnt + e0);
  });
}

hipError_t launch_select_offsets(hipStream_t st, const int32_t* cnt, int64_t n_events, int64_t* off) {
  hipLaunchKernelGGL(k_select_offsets, dim3(1), dim3(1024), 0, st, cnt, n_events, off);
  return hipGetLastError();
}

hipError_t launch_select_write(hipStream_t st, const float* feat, int ldf, const int64_t* off,
                               const int64_t* off_out, int64_t n_events, const uint8_t* keep,
                               float* out) {
  if (n_events <= 0) return hipSuccess;
  if (n_events > 0x7fffffff) return hipErrorInvalidValue;
  return event_parts(n_events, [&](int64_t e0, unsigned n) {
    hipLaunchKernelGGL(k_select_write, dim3(n), dim3(256), 0, st, feat, ldf, off + e0, off_out + e0, keep,
                       out);
  });
}

}  // namespace fmd
