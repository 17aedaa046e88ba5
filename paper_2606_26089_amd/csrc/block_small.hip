// Fused BF16 block kernels (d = 256, 8 heads of 32) for calls whose rows do not fill the chip:
// the same three kernels as block_bf16.hip, and bitwise the same rows, split for latency.
//
// A throughput workgroup takes 64 rows through a whole block segment with one wave per SIMD;
// with fewer row tiles than CUs the rest of the chip idles and that one serial chain is the
// call's time. Here a workgroup takes 32 TM rows with eight waves, wave w holding columns
// [32w, 32w + 32), so each wave has a quarter (TM = 1) of the chain and the two waves of a SIMD
// hide each other's waits. What bounds it then is the weight stream: a segment's weights pass
// through one CU at about 64 bytes per cycle, so every product phase is 16 fragments per wave,
// all 16 in flight (each consumed fragment is replaced by the next phase's at once). Per launch
// with 105 rows: MLP 33 -> 21 us (10 of them the stream), OQC 10.8 -> 6.5, embedding + QKV 15 ->
// 9.5; an evaluation of 4,103 rows 406 -> 295 us, of 14,276 (64-row tiles) 510 -> 465.
//
// LayerNorm: the rows go through LDS once in FP32 and 16 lanes take each row, lane j the
// columns 16 k + j. Sums are formed in the order of the throughput kernels (partial sums over
// their waves' columns by the same exchange tree, then the partials in wave order), so a row's
// bits do not depend on the form that computed it.
#include "block_common.h"

namespace fmd {
namespace {

constexpr int kPhase = 16;            // fragments of a product phase per wave
constexpr int kLdX = kD + 16;         // FP32 row pitch: four rows x 16 lanes hit 64 banks
constexpr int kChunk = 256;           // MLP hidden units per chunk (32 per wave)
constexpr int kChunks = 4 * kD / kChunk;
static_assert(kKs == kPhase && kChunk / 16 == kPhase, "one ring per phase");

__device__ __forceinline__ void fill16(u32x4 (&ring)[kPhase], const u32x4* __restrict__ src,
                                       int lane) {
#pragma unroll
  for (int k = 0; k < kPhase; ++k) ring[k] = src[k * 64 + lane];
}

// acc[mi] += tile rows [32 mi, 32 mi + 32) x the 16 fragments in the ring; with NEXT each
// fragment is replaced by the next phase's as it is used. beside(k) is work for the vector ALUs
// next to K step k.
template <bool NEXT, int TM, typename F>
__device__ __forceinline__ void phase16(f32x16 (&acc)[TM], const bf16* __restrict__ tile,
                                        u32x4 (&ring)[kPhase], const u32x4* __restrict__ next,
                                        int lane, F&& beside) {
  asm volatile("" ::: "memory");   // the tile's reads stay in their phase
  const bf16* arow = tile + (lane & 31) * kLdA + (lane >> 5) * 8;
#pragma unroll
  for (int k = 0; k < kPhase; ++k) {
    bf16x8 a[TM];
#pragma unroll
    for (int mi = 0; mi < TM; ++mi) a[mi] = *(const bf16x8*)(arow + mi * 32 * kLdA + k * 16);
    const bf16x8 b = as_bf16x8(ring[k]);
    if constexpr (NEXT) ring[k] = next[k * 64 + lane];
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
      acc[mi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[mi], b, acc[mi], 0, 0, 0);
    beside(k);
    __builtin_amdgcn_sched_barrier(kKeepLoadsAndMfma);   // loads stay 16 fragments ahead
  }
}

template <bool NEXT, int TM>
__device__ __forceinline__ void phase16(f32x16 (&acc)[TM], const bf16* __restrict__ tile,
                                        u32x4 (&ring)[kPhase], const u32x4* __restrict__ next,
                                        int lane) {
  phase16<NEXT>(acc, tile, ring, next, lane, [](int) {});
}

template <int TM>
__device__ __forceinline__ void acc_to_x(const f32x16 (&acc)[TM], float* __restrict__ X, int col,
                                         int lane) {
#pragma unroll
  for (int mi = 0; mi < TM; ++mi)
#pragma unroll
    for (int r = 0; r < 16; ++r) X[acc_row(mi, r, lane) * kLdX + col] = acc[mi][r];
}

template <int CTRL>
__device__ __forceinline__ float dpp_of(float v) {
  return __builtin_amdgcn_update_dpp(0.f, v, CTRL, 0xF, 0xF, false);
}

// Sum over the 16 lanes of a row group, the same in each of them: the exchange tree of the
// throughput kernels' reductions over lane bits 3..0.
__device__ __forceinline__ float row16_sum(float v) {
#pragma clang fp contract(off)
  v = v + dpp_of<kDppRor8>(v);
  v = v + dpp_of<kDppHalfMirror>(v);
  v = v + dpp_of<kDppXor2>(v);
  v = v + dpp_of<kDppXor1>(v);
  return v;
}

// This lane's share of partial sum q of P over a row, value x[k] of column 16 k + j: P = 4 is
// the order of the four-wave kernels (columns 64 q + c and 64 q + 32 + c first), P = 8 of the
// eight-wave ones (32 columns per partial).
template <int P>
__device__ __forceinline__ float share(const float (&x)[16], int q) {
#pragma clang fp contract(off)
  if constexpr (P == 4)
    return (x[4 * q] + x[4 * q + 2]) + (x[4 * q + 1] + x[4 * q + 3]);
  else
    return x[2 * q] + x[2 * q + 1];
}

template <int P>
__device__ __forceinline__ float row_sum(const float (&x)[16]) {
#pragma clang fp contract(off)
  float t = 0.f;
#pragma unroll
  for (int q = 0; q < P; ++q) t += row16_sum(share<P>(x, q));
  return t;
}

// LayerNorm statistics (mean, 1/sqrt(biased variance + eps)) of the row whose columns
// 16 k + j this lane holds.
template <int P>
__device__ __forceinline__ float2 row_stats16(const float (&x)[16]) {
#pragma clang fp contract(off)
  const float mu = row_sum<P>(x) * (1.0f / kD);
  float d[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const float dv = x[k] - mu;
    d[k] = dv * dv;
  }
  const float rs = rsqrtf(row_sum<P>(d) * (1.0f / kD) + kLnEps);
  return make_float2(mu, rs);
}

__device__ __forceinline__ void read16(float (&x)[16], const float* __restrict__ p, int j) {
#pragma unroll
  for (int k = 0; k < 16; ++k) x[k] = p[16 * k + j];
}

// Column parameters of up to two LayerNorms in LDS (each lane needs 16 columns of both).
struct SmallParams {
  float g[2][kD], s[2][kD];
};

// A (BF16, pitch kLdA) = LayerNorm of the rows in X with gain g and shift s, 16 lanes a row.
template <int P, int TM>
__device__ __forceinline__ void ln_rows(const float* __restrict__ X, bf16* __restrict__ A,
                                        const float* __restrict__ g, const float* __restrict__ s,
                                        float2* __restrict__ stats_out, int64_t m0, int tid) {
  const int j = tid & 15;
#pragma unroll
  for (int m = 0; m < TM; ++m) {
    const int row = (tid >> 4) + 32 * m;
    float x[16];
    read16(x, X + row * kLdX, j);
    const float2 st = row_stats16<P>(x);
    if (stats_out && j == 0) stats_out[m0 + row] = st;
#pragma unroll
    for (int k = 0; k < 16; ++k)
      A[row * kLdA + 16 * k + j] = (bf16)((x[k] - st.x) * st.y * g[16 * k + j] + s[16 * k + j]);
  }
}

template <int TM>
__device__ __forceinline__ void store_h(const f32x16 (&acc)[TM], float* __restrict__ H, int64_t m0,
                                        int col, int lane) {
  const RowIo<float, kD> io(H, m0, col, lane);
#pragma unroll
  for (int mi = 0; mi < TM; ++mi)
#pragma unroll
    for (int r = 0; r < 16; ++r) *io.at(mi, r) = acc[mi][r];
}

// head-major BF16 plane of 32 columns
template <int TM>
__device__ __forceinline__ void store_plane(const f32x16 (&acc)[TM], bf16* __restrict__ plane,
                                            int64_t m0, int lane) {
  const RowIo<bf16, kDh> io(plane, m0, lane & 31, lane);
#pragma unroll
  for (int mi = 0; mi < TM; ++mi)
#pragma unroll
    for (int r = 0; r < 16; ++r) *io.at(mi, r) = (bf16)acc[mi][r];
}

template <int TM>
__device__ __forceinline__ void fill_acc(f32x16 (&acc)[TM], float v) {
#pragma unroll
  for (int mi = 0; mi < TM; ++mi)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[mi][r] = v;
}

// First row of this workgroup: a map lists 64-row tiles, 2 / TM workgroups each.
template <int TM>
__device__ __forceinline__ int64_t small_first_row(const RowMap& rm) {
  if (!rm.tiles) return (int64_t)blockIdx.x * (32 * TM);
  constexpr int kPer = 2 / TM;
  return (int64_t)rm.tiles[blockIdx.x / kPer] * 64 + (int64_t)(blockIdx.x % kPer) * 32;
}

// The three slabs of [Q | K | V] from the LayerNorm tile A; the ring holds slab 0.
template <int TM>
__device__ __forceinline__ void qkv_slabs(f32x16 (&acc)[TM], const bf16* __restrict__ A,
                                          u32x4 (&ring)[kPhase], const u32x4* __restrict__ wf,
                                          const float (&b)[3], bf16* __restrict__ qkv,
                                          int64_t plane, int64_t m0, int w, int lane) {
#pragma unroll
  for (int slab = 0; slab < 3; ++slab) {
    fill_acc(acc, b[slab]);
    if (slab < 2)
      phase16<true>(acc, A, ring, wf + (slab + 1) * kWaves * kKs * 64, lane);
    else
      phase16<false>(acc, A, ring, wf, lane);
    store_plane(acc, qkv + (int64_t)(slab * kWaves + w) * plane, m0, lane);
  }
}

}  // namespace

template <int TM, bool EMBED>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_small_qkv(
    const float* __restrict__ H, const float* __restrict__ g, const float* __restrict__ s,
    const u32x4* __restrict__ Wf, const float* __restrict__ bias, bf16* __restrict__ qkv,
    EmbedRows em, RowMap rm) {
  constexpr int ROWS = 32 * TM;
  __shared__ __attribute__((aligned(16))) bf16 A[ROWS * kLdA];
  __shared__ __attribute__((aligned(16))) float X[ROWS * kLdX];
  __shared__ SmallParams prm;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t m0 = small_first_row<TM>(rm), plane = rm.Mp * kDh;
  const int col = w * 32 + (lane & 31);
  const u32x4* wf = Wf + w * kKs * 64;
  float b[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) b[i] = bias[i * kD + col];
  if (tid < kD) {
    prm.g[0][tid] = g[tid];
    prm.s[0][tid] = s[tid];
  }
  f32x16 acc[TM];
  u32x4 ring[kPhase];
  if constexpr (EMBED) {
    static_assert(ROWS * kEmbLd * 4 <= ROWS * kLdA * 2, "staging fits the A tile");
    float* xt = reinterpret_cast<float*>(A);
    for (int i = tid; i < ROWS * kEmbLd / 4; i += kThreads)
      *(float4*)&xt[4 * i] = *(const float4*)&em.xs[m0 * kEmbLd + 4 * i];
    float wv[kEmbF9];
#pragma unroll
    for (int k = 0; k < kEmbF9; ++k) wv[k] = em.W[k * kD + col];
    const float t0 = stage_row(em.temb, em.ctl, kD)[col];
    fill16(ring, wf, lane);
    __syncthreads();
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = acc_row(mi, r, lane);
        const float* x = &xt[row * kEmbLd];
        const float4 x0 = *(const float4*)x, x1 = *(const float4*)(x + 4);
        const float xv[kEmbF9] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w, x[8]};
        float v = t0;
#pragma unroll
        for (int k = 0; k < kEmbF9; ++k) v = fmaf(xv[k], wv[k], v);
        acc[mi][r] = m0 + row < em.T ? v : 0.f;
      }
    store_h(acc, em.H, m0, col, lane);
  } else {
    fill16(ring, wf, lane);
    const RowIo<float, kD> io(H, m0, col, lane);
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][r] = *io.at(mi, r);
  }
  acc_to_x(acc, X, col, lane);
  __syncthreads();   // also: the staged state rows are consumed
  ln_rows<8, TM>(X, A, prm.g[0], prm.s[0], nullptr, m0, tid);
  __syncthreads();
  qkv_slabs(acc, A, ring, wf, b, qkv, plane, m0, w, lane);
}

template <int TM>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_small_oqc(
    const bf16* __restrict__ att, const u32x4* __restrict__ Wf_o, const float* __restrict__ b_o,
    float* __restrict__ H, const float* __restrict__ g, const float* __restrict__ s,
    const u32x4* __restrict__ Wf_qc, const float* __restrict__ b_qc, bf16* __restrict__ qc,
    RowMap rm) {
  constexpr int ROWS = 32 * TM;
  __shared__ __attribute__((aligned(16))) bf16 A[ROWS * kLdA];
  __shared__ __attribute__((aligned(16))) float X[ROWS * kLdX];
  __shared__ SmallParams prm;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t m0 = small_first_row<TM>(rm), plane = rm.Mp * kDh;
  const int col = w * 32 + (lane & 31);
  const u32x4* wq = Wf_qc + w * kKs * 64;
  const float bo = b_o[col], bq = b_qc[col];
  tile_hm_to_lds<ROWS, kThreads>(A, att, plane, m0, tid);
  f32x16 acc[TM];
  {
    const RowIo<float, kD> io(H, m0, col, lane);
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][r] = *io.at(mi, r) + bo;
  }
  u32x4 ring[kPhase];
  fill16(ring, Wf_o + w * kKs * 64, lane);
  if (tid < kD) {
    prm.g[0][tid] = g[tid];
    prm.s[0][tid] = s[tid];
  }
  __syncthreads();
  phase16<true>(acc, A, ring, wq, lane);
  acc_to_x(acc, X, col, lane);
  store_h(acc, H, m0, col, lane);
  __syncthreads();
  ln_rows<8, TM>(X, A, prm.g[0], prm.s[0], nullptr, m0, tid);
  __syncthreads();
  fill_acc(acc, bq);
  phase16<false>(acc, A, ring, wq, lane);
  store_plane(acc, qc + (int64_t)w * plane, m0, lane);
}

namespace {
constexpr int kLdC8 = kChunk + 16;    // bytes per row of an FP8 hidden chunk
constexpr int kDn8 = kChunk / 64;     // 64-deep K steps of a chunk
}  // namespace

template <int TM, int TAIL, bool F8>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_small_mlp(
    const bf16* __restrict__ att, const u32x4* __restrict__ Wf_oc, const float* __restrict__ b_oc,
    float* __restrict__ H, const float* __restrict__ g, const float* __restrict__ s,
    const u32x4* __restrict__ Wf_up, const float* __restrict__ b_up,
    const u32x4* __restrict__ Wf_dn, const float* __restrict__ b_dn,
    float2* __restrict__ stats_out, NextQkv nq, NextHead nh, Mlp8 f8, RowMap rm) {
  constexpr bool QKV = TAIL == kTailQkv, HEAD = TAIL == kTailHead;
  constexpr int ROWS = 32 * TM;
  __shared__ __attribute__((aligned(16))) bf16 A[ROWS * kLdA];
  // the FP32 rows of a LayerNorm and the two hidden chunks are never live together
  union Scratch {
    float X[ROWS * kLdX];
    bf16 Hc[2][ROWS * kLdA];
  };
  __shared__ __attribute__((aligned(16))) Scratch sc;
  __shared__ SmallParams prm;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t m0 = small_first_row<TM>(rm), plane = rm.Mp * kDh;
  const int col = w * 32 + (lane & 31);
  auto up_c = [&](int c) { return Wf_up + (8 * c + w) * kKs * 64; };
  auto dn_c = [&](int c) { return Wf_dn + (w * 4 * kD / 16 + c * kPhase) * 64; };
  const u32x4* wqkv = QKV ? nq.Wf + w * kKs * 64 : nullptr;
  tile_hm_to_lds<ROWS, kThreads>(A, att, plane, m0, tid);
  f32x16 acc[TM];
  {
    const float bv = b_oc[col];
    const RowIo<float, kD> io(H, m0, col, lane);
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][r] = *io.at(mi, r) + bv;
  }
  u32x4 ring[kPhase];
  fill16(ring, Wf_oc + w * kKs * 64, lane);
  if (tid < kD) {
    prm.g[0][tid] = g[tid];
    prm.s[0][tid] = s[tid];
    if constexpr (QKV || HEAD) {
      prm.g[1][tid] = QKV ? nq.g[tid] : nh.g[tid];
      prm.s[1][tid] = QKV ? nq.s[tid] : nh.s[tid];
    }
  }
  float bq[3] = {0.f, 0.f, 0.f};
  if constexpr (QKV) {
#pragma unroll
    for (int i = 0; i < 3; ++i) bq[i] = nq.bias[i * kD + col];
  }
  const float bd = b_dn[col];
  __syncthreads();
  phase16<!F8>(acc, A, ring, F8 ? nullptr : up_c(0), lane);
  acc_to_x(acc, sc.X, col, lane);
  __syncthreads();
  if constexpr (!F8) {
    ln_rows<4, TM>(sc.X, A, prm.g[0], prm.s[0], nullptr, m0, tid);
    __syncthreads();
    f32x16 h2[2][TM];
    // GELU of values [v0, v0 + n) of a chunk's products (value v: row block v / 16, register
    // v % 16) into its hidden buffer
    auto gelu = [&](const f32x16 (&h)[TM], int v0, int n, float bu, bf16* hb) {
#pragma unroll
      for (int q = 0; q < n; ++q) {
        const int v = v0 + q, mi = v >> 4, r = v & 15;
        hb[acc_row(mi, r, lane) * kLdA + col] = (bf16)gelu_as(h[mi][r], bu);
      }
    };
    constexpr int kHalf = 8 * TM;    // values of half a chunk
    // halves spread over a phase's 16 K steps: TM = 1 one value every second step
    auto gelu_step = [&](const f32x16 (&h)[TM], int v0, int k, float bu, bf16* hb) {
      if constexpr (TM == 1) {
        if (k % 2 == 0) gelu(h, v0 + k / 2, 1, bu, hb);
      } else {
        gelu(h, v0 + k * (kHalf / kPhase), kHalf / kPhase, bu, hb);
      }
    };
    float bu = kGeluU * b_up[col];
    fill_acc(h2[0], 0.f);
    phase16<true>(h2[0], A, ring, up_c(1), lane);
    gelu(h2[0], 0, kHalf, bu, sc.Hc[0]);
    // chunk c: [up-projection c + 1 | GELU c, second half] -> barrier -> [down-projection c |
    // GELU c + 1, first half]
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      const bool more = c + 1 < kChunks;
      const float bun = more ? kGeluU * b_up[(c + 1) * kChunk + col] : 0.f;
      f32x16 (&h)[TM] = h2[c & 1];
      f32x16 (&hn)[TM] = h2[(c + 1) & 1];
      if (more) {
        fill_acc(hn, 0.f);
        phase16<true>(hn, A, ring, dn_c(c), lane,
                      [&](int k) { gelu_step(h, kHalf, k, bu, sc.Hc[c & 1]); });
      } else {
        gelu(h, kHalf, kHalf, bu, sc.Hc[c & 1]);
      }
      __syncthreads();
      if (c + 2 < kChunks)
        phase16<true>(acc, sc.Hc[c & 1], ring, up_c(c + 2), lane,
                      [&](int k) { gelu_step(hn, 0, k, bun, sc.Hc[(c + 1) & 1]); });
      else if (more)
        phase16<true>(acc, sc.Hc[c & 1], ring, dn_c(c + 1), lane,
                      [&](int k) { gelu_step(hn, 0, k, bun, sc.Hc[(c + 1) & 1]); });
      else if constexpr (QKV)
        phase16<true>(acc, sc.Hc[c & 1], ring, wqkv, lane);
      else
        phase16<false>(acc, sc.Hc[c & 1], ring, wqkv, lane);
      bu = bun;
    }
  } else {
    // FP8 operands for W_up and W_dn: the LayerNorm tile and the hidden chunks as e4m3 bytes,
    // the residual rows in W_dn's scaled domain
    uint8_t* A8 = reinterpret_cast<uint8_t*>(A);
    uint8_t* H8 = reinterpret_cast<uint8_t*>(sc.Hc);
    i32x8 fu[kKs8], fd[kDn8];
#pragma unroll
    for (int ks = 0; ks < kKs8; ++ks) fu[ks] = f8.up[(w * kKs8 + ks) * 64 + lane];
    {
      const int j = tid & 15;
#pragma unroll
      for (int m = 0; m < TM; ++m) {
        const int row = (tid >> 4) + 32 * m;
        float x[16];
        read16(x, sc.X + row * kLdX, j);
        const float2 st = row_stats16<4>(x);
#pragma unroll
        for (int k = 0; k < 16; ++k) {
          const int c = 16 * k + j;
          A8[row * kLdA8 + c] =
              (uint8_t)to_fp8((x[k] - st.x) * st.y * prm.g[0][c] + prm.s[0][c]);
        }
      }
      const float sd = f8.dn_scale[col];
#pragma unroll
      for (int mi = 0; mi < TM; ++mi)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[mi][r] *= sd;
    }
    __syncthreads();
#pragma unroll 1
    for (int c = 0; c < kChunks; ++c) {
      const float ui = f8.up_inv[c * kChunk + col], bu = kGeluU * b_up[c * kChunk + col];
#pragma unroll
      for (int ks = 0; ks < kDn8; ++ks)
        fd[ks] = f8.dn[(w * (4 * kD / 64) + c * kDn8 + ks) * 64 + lane];
      asm volatile("" ::: "memory");
      f32x16 h[TM];
      fill_acc(h, 0.f);
#pragma unroll
      for (int ks = 0; ks < kKs8; ++ks)
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
          h[mi] = mfma_f8(lds_frag8(A8, kLdA8, 32 * mi + (lane & 31), ks, lane), fu[ks], h[mi]);
      if (c + 1 < kChunks) {
#pragma unroll
        for (int ks = 0; ks < kKs8; ++ks)
          fu[ks] = f8.up[((8 * (c + 1) + w) * kKs8 + ks) * 64 + lane];
      }
      uint8_t* hb = H8 + (c & 1) * (ROWS * kLdC8);
#pragma unroll
      for (int mi = 0; mi < TM; ++mi)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          hb[acc_row(mi, r, lane) * kLdC8 + col] = (uint8_t)to_fp8(gelu_as(h[mi][r] * ui, bu));
      __syncthreads();
#pragma unroll
      for (int ks = 0; ks < kDn8; ++ks)
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
          acc[mi] = mfma_f8(lds_frag8(hb, kLdC8, 32 * mi + (lane & 31), ks, lane), fd[ks], acc[mi]);
    }
    if constexpr (QKV) fill16(ring, wqkv, lane);
    const float sdi = f8.dn_inv[col];
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][r] *= sdi;
  }
#pragma unroll
  for (int mi = 0; mi < TM; ++mi)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[mi][r] += bd;
  if constexpr (!HEAD) store_h(acc, H, m0, col, lane);
  __syncthreads();   // every wave is past its last read of the hidden chunks (and of A)
  acc_to_x(acc, sc.X, col, lane);
  float* wt = reinterpret_cast<float*>(A);   // head weights [9][256], over the LN3 tile
  constexpr int kF = 9;
  if constexpr (HEAD) {
    for (int i = tid; i < kF * kD / 4; i += kThreads) *(float4*)&wt[4 * i] = *(const float4*)&nh.Wt[4 * i];
  }
  __syncthreads();
  if constexpr (TAIL == kTailStats) {
    const int j = tid & 15;
#pragma unroll
    for (int m = 0; m < TM; ++m) {
      const int row = (tid >> 4) + 32 * m;
      float x[16];
      read16(x, sc.X + row * kLdX, j);
      const float2 st = row_stats16<4>(x);
      if (stats_out && j == 0) stats_out[m0 + row] = st;
    }
  } else if constexpr (QKV) {
    ln_rows<4, TM>(sc.X, A, prm.g[1], prm.s[1], stats_out, m0, tid);
    __syncthreads();
    qkv_slabs(acc, A, ring, wqkv, bq, nq.qkv, plane, m0, w, lane);
  } else {
    const OdeArgs& od = nh.ode;
    const int j = tid & 15;
    const OdeStage os = ode_stage(od);
    float* out = os.out;
    ode_next_stage(od);
#pragma unroll
    for (int m = 0; m < TM; ++m) {
      const int row = (tid >> 4) + 32 * m;
      float y[16];
      read16(y, sc.X + row * kLdX, j);
      const float2 st = row_stats16<4>(y);
#pragma unroll
      for (int k = 0; k < 16; ++k)
        y[k] = fmaf((y[k] - st.x) * st.y, prm.g[1][16 * k + j], prm.s[1][16 * k + j]);
      float v = 0.f;
#pragma unroll
      for (int f = 0; f < kF; ++f) {
        const float* wf = wt + f * kD + j;
        float p[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          // columns 64 q + c and 64 q + 32 + c in one multiply-add each, as the four-wave head
          const float lo = fmaf(y[4 * q + 2], wf[64 * q + 32], y[4 * q] * wf[64 * q]);
          const float hi = fmaf(y[4 * q + 3], wf[64 * q + 48], y[4 * q + 1] * wf[64 * q + 16]);
          p[q] = row16_sum(lo + hi);
        }
        const float t = ((p[0] + p[1]) + p[2]) + p[3] + nh.b[f];
        v = j == f ? t : v;
      }
      const int64_t r = m0 + row;
      if (j < kF && r < od.m_valid) {
        const int64_t o = r * od.ldx + j;
        if (od.tok_event) {
          const StageDesc sd = od.desc[od.tok_event[r]];
          ode_update(sd.mode, sd.h, v, od.x + o, od.acc + o, od.xs + o,
                     out && sd.write_out ? out + r * od.ldo + j : nullptr);
        } else {
          ode_update(os.mode, os.h, v, od.x + o, od.acc + o, od.xs + o,
                     out ? out + r * od.ldo + j : nullptr);
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------------

static bool small_grid(int64_t Mp, int rows, const int32_t* tiles, int64_t n_tiles, unsigned* grid) {
  if ((rows != 32 && rows != 64) || Mp % 64 || (tiles && n_tiles > Mp / 64)) return false;
  *grid = (unsigned)(tiles ? n_tiles * (64 / rows) : Mp / rows);
  return true;
}

hipError_t launch_small_qkv(hipStream_t st, int64_t Mp, int rows, const float* H, const float* g,
                            const float* s, const void* Wf, const float* bias, void* qkv,
                            const int32_t* tiles, int64_t n_tiles) {
  unsigned grid = 0;
  if (!small_grid(Mp, rows, tiles, n_tiles, &grid)) return hipErrorInvalidValue;
  if (grid == 0) return hipSuccess;
  const RowMap rm{tiles, Mp};
  auto* k = rows == 32 ? k_small_qkv<1, false> : k_small_qkv<2, false>;
  hipLaunchKernelGGL(k, dim3(grid), dim3(kThreads), 0, st, H, g, s, (const u32x4*)Wf, bias,
                     (bf16*)qkv, EmbedRows{}, rm);
  return hipGetLastError();
}

hipError_t launch_small_embed_qkv(hipStream_t st, int64_t Mp, int rows, const float* xs, int ldx,
                                  int f, int64_t T, const float* temb, StageCtl* ctl,
                                  const float* W_xin, float* H, const float* g, const float* s,
                                  const void* Wf, const float* bias, void* qkv) {
  unsigned grid = 0;
  if (!small_grid(Mp, rows, nullptr, 0, &grid) || ldx != kEmbLd || f != kEmbF9 || T > Mp)
    return hipErrorInvalidValue;
  if (grid == 0) return hipSuccess;
  const EmbedRows em{xs, T, temb, ctl, W_xin, H};
  auto* k = rows == 32 ? k_small_qkv<1, true> : k_small_qkv<2, true>;
  hipLaunchKernelGGL(k, dim3(grid), dim3(kThreads), 0, st, nullptr, g, s, (const u32x4*)Wf, bias,
                     (bf16*)qkv, em, RowMap{nullptr, Mp});
  return hipGetLastError();
}

hipError_t launch_small_oqc(hipStream_t st, int64_t Mp, int rows, const void* att, const void* Wf_o,
                            const float* b_o, float* H, const float* g, const float* s,
                            const void* Wf_qc, const float* b_qc, void* qc, const int32_t* tiles,
                            int64_t n_tiles) {
  unsigned grid = 0;
  if (!small_grid(Mp, rows, tiles, n_tiles, &grid)) return hipErrorInvalidValue;
  if (grid == 0) return hipSuccess;
  auto* k = rows == 32 ? k_small_oqc<1> : k_small_oqc<2>;
  hipLaunchKernelGGL(k, dim3(grid), dim3(kThreads), 0, st, (const bf16*)att, (const u32x4*)Wf_o,
                     b_o, H, g, s, (const u32x4*)Wf_qc, b_qc, (bf16*)qc, RowMap{tiles, Mp});
  return hipGetLastError();
}

hipError_t launch_small_mlp(hipStream_t st, int64_t Mp, int rows, const FusedMlpArgs& a) {
  unsigned grid = 0;
  if (!small_grid(Mp, rows, a.tiles, a.n_tiles, &grid) || !fused_mlp_args(a)) return hipErrorInvalidValue;
  if (grid == 0) return hipSuccess;
  const MlpTailArgs t = mlp_tail_args(a);
#define FMD_SMALL_TAIL(TM, F8)                                            \
  (a.qkv ? k_small_mlp<TM, kTailQkv, F8>                                  \
         : a.head ? k_small_mlp<TM, kTailHead, F8> : k_small_mlp<TM, kTailStats, F8>)
  auto* k = rows == 32 ? (a.fp8 ? FMD_SMALL_TAIL(1, true) : FMD_SMALL_TAIL(1, false))
                       : (a.fp8 ? FMD_SMALL_TAIL(2, true) : FMD_SMALL_TAIL(2, false));
#undef FMD_SMALL_TAIL
  hipLaunchKernelGGL(k, dim3(grid), dim3(kThreads), 0, st, (const bf16*)a.att,
                     (const u32x4*)a.Wf_oc, a.b_oc, a.H, a.g, a.s, (const u32x4*)a.Wf_up, a.b_up,
                     (const u32x4*)a.Wf_dn, a.b_dn, a.stats_out, t.nq, t.nh, t.f8, RowMap{a.tiles, Mp});
  return hipGetLastError();
}

}  // namespace fmd
