// FP32 products of the velocity network on the BF16 matrix cores (gfx950), for d_model <= 256.
//
// C[M, N] = epi(pro(A)[M, K] W[K, N] + b) as launch_gemm, with FP32 operands and results. An
// FP32 value is the sum of three BF16 values, x = hi + mid + lo: hi its top 8 significand bits
// (truncated, so it is finite whenever x is), mid and lo the remainders rounded to nearest, with
// a rest below 2^-24 |x|. A product is the sum of the six partial products down to 2^-16 of it
// (hi hi, hi mid, mid hi, mid mid, hi lo, lo hi; the ones left out are below 2^-23 and of either
// sign), each exact in the matrix core's FP32 accumulator. Six BF16 instructions take 192 cycles
// for what the FP32 instruction takes 512; hi hi is accumulated apart from the five small terms,
// one rounding per 16 k.
//
// A workgroup of eight waves takes 32 TM rows and a range of 32-column blocks, one per wave at a
// time. The rows are read once, normalised if asked (16 bytes a lane, a row by 16, 32 or 64
// lanes, statistics from the registers) and written to LDS as three BF16 planes; the weights
// stream from L2 as packed fragments of three planes, four K steps in flight, as in the BF16
// block kernels. A K above 256 (the MLP down-projection) goes in panels of 256 columns, the next
// panel's rows in registers while the current one is multiplied. Every output element is formed
// in the same order whatever the tile, so a row's bits do not depend on the batch around it.
//
// Bound: the power the matrix cores may draw (six instructions a product; a library BF16 GEMM
// reaches 1205 TFLOP/s on this card): the clock falls as the instructions get denser (cross K/V:
// 1.79 GHz at 47% matrix busy, 1.64 GHz at 60%). 448,552 rows, d = 256, against the GEMMs on the
// FP32 instruction before: up 2466 -> 1405 us (1005 TFLOP/s of BF16 instructions), down 2392 -> 1346
// (1049), QKV 1601 -> 1053 (1006), projections 968 -> 411 (their row statistics went too), cross
// K/V 6590 -> 4080. 14,276 rows (one tile per CU, so its chain): down 177 -> 47 us, up 98 -> 50,
// projections 71 -> 17. Of that, operand reads spread over the products of the step before (left
// alone, the compiler reads each right before its product), K steps unrolled and the next panel
// split beside the products gave 3 to 17% a kernel. Vector instructions beside the products cost
// matrix issue (addresses as 64-bit vectors and a branching erf: up 1684, down 1517 us), hence the
// uniform addresses and the GELU below. Error of one velocity evaluation of the base network on
// 4096 events against 64 bits (2-norm): 6.3e-7 -> 3.3e-7.
//
// Weight layout (launch_pack_split): [N/32][K/16][3 planes][64 lanes][8], lane l of fragment
// (nb, ks) holding W[16 ks + 8 (l/32) + j][32 nb + l%32].
#include "split_common.h"

namespace fmd {
namespace {

constexpr int kNw = 8;                 // waves
constexpr int kNt = 64 * kNw;
constexpr int kPanel = 256;            // K columns in LDS at a time
constexpr int kLdP = kPanel + 8;       // LDS pitch (bf16) of a plane row
// sched_group_barrier instruction classes
constexpr int kSchedValu = 0x002, kSchedMfma = 0x008, kSchedVmemRead = 0x020, kSchedDsRead = 0x100;

}  // namespace

// SRC: where the rows come from. EMBED: row r = base + sum_k x[r][k] Win[k] over 9 features
// (base first, then the features in order), rows at or past T zero; optionally stored to H.
enum SplitSrc { SRC_ROWS = 0, SRC_LN = 1, SRC_EMBED_LN = 2 };

// NKS: K steps of 16 (of a panel, if MULTI: K in several panels, a panel's rows in registers while
// the one before is multiplied, and N at most one pass).
template <int TM, int SRC, int EPI, int NKS, bool MULTI>
__device__ __forceinline__ void split_body(const SplitArgs& p) {
  constexpr int ROWS = 32 * TM;
  constexpr int KL = NKS <= 4 ? 16 : NKS <= 8 ? 32 : 64;   // lanes that hold one row, 4 columns each
  constexpr int RPI = 64 / KL;                       // rows of one wave-wide load
  constexpr int NI = (ROWS / kNw + RPI - 1) / RPI;   // loads per lane and panel
  constexpr bool LN = SRC != SRC_ROWS;
  constexpr int kDepth = 4;                          // K steps of weight fragments in flight
  static_assert(!MULTI || (NKS == kPanel / 16 && NI <= NKS / 2 && EPI == EPI_RESID), "one pass");
  __shared__ __attribute__((aligned(16))) bf16 P[3][ROWS * kLdP];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t m0 = (int64_t)blockIdx.x * ROWS;
  const int nb0 = blockIdx.y * p.nb_per, nb1 = min(nb0 + p.nb_per, p.N / 32);
  constexpr int kp = 16 * NKS;
  const int n_panels = MULTI ? p.K / kPanel : 1, nks = p.K / 16;
  // staging: lane group lg of this wave takes rows row_of(i), lane gl of the group columns c4 ..
  const int gl = lane % KL, lg = lane / KL, c4 = 4 * gl;
  const bool in_row = c4 < kp;
  auto row_of = [&](int i) { return w * (ROWS / kNw) + i * RPI + lg; };
  float4 v[NI];

  auto load = [&](int panel) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (in_row && (RPI * NI * kNw == ROWS || row_of(i) < (w + 1) * (ROWS / kNw)))
        v[i] = *(const float4*)(p.A + (m0 + row_of(i)) * p.lda + panel * kPanel + c4);
    }
  };
  bf16x4 pl[NI][3];
  auto stage = [&]() {   // split rows -> LDS planes
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      if (!in_row || !(RPI * NI * kNw == ROWS || row_of(i) < (w + 1) * (ROWS / kNw))) continue;
#pragma unroll
      for (int q = 0; q < 3; ++q) *(bf16x4*)&P[q][row_of(i) * kLdP + c4] = pl[i][q];
    }
  };

  // weight stream of this wave's first column block, ahead of the rows: a wave-uniform address
  // (3 KB a K step) and one lane offset, so that the loads cost no vector instructions
  constexpr int kStep = 3 * 64 * 16;                 // bytes of a K step
  const char* const wbase = (const char*)p.Wf;
  const int64_t block_bytes = (int64_t)nks * kStep;
  const uint32_t l16 = lane * 16;
  u32x4 ring[kDepth][3];
  if (nb0 + w < nb1) {
    const char* f = wbase + (nb0 + w) * block_bytes;
#pragma unroll
    for (int s = 0; s < kDepth; ++s)
#pragma unroll
      for (int q = 0; q < 3; ++q) ring[s][q] = *(const u32x4*)(f + s * kStep + q * 1024 + l16);
  }
  if constexpr (SRC == SRC_EMBED_LN) {
    float4 wk[9];
#pragma unroll
    for (int k = 0; k < 9; ++k)
      wk[k] = in_row ? *(const float4*)(p.Win + k * p.K + c4) : make_float4(0.f, 0.f, 0.f, 0.f);
    const float* base = stage_row(p.base, p.ctl, p.K);
    const float4 b4 = in_row ? *(const float4*)(base + c4) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int64_t r = m0 + row_of(i);
      v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (r < p.T && (RPI * NI * kNw == ROWS || row_of(i) < (w + 1) * (ROWS / kNw))) {
        v[i] = b4;
        if (p.tok_event && in_row)   // the event's own base row
          v[i] = *(const float4*)(p.base + (int64_t)p.tok_event[r] * p.K + c4);
#pragma unroll
        for (int k = 0; k < 9; ++k) {
          const float x = p.A[r * p.lda + k];
          v[i].x = fmaf(x, wk[k].x, v[i].x);
          v[i].y = fmaf(x, wk[k].y, v[i].y);
          v[i].z = fmaf(x, wk[k].z, v[i].z);
          v[i].w = fmaf(x, wk[k].w, v[i].w);
        }
      }
      if (p.H && blockIdx.y == 0 && in_row &&
          (RPI * NI * kNw == ROWS || row_of(i) < (w + 1) * (ROWS / kNw)))
        *(float4*)(p.H + r * p.K + c4) = v[i];
    }
  } else {
    load(0);
  }
  if constexpr (LN) {
    const float inv = 1.0f / (float)p.K;
    const float4 g4 = in_row ? *(const float4*)(p.g + c4) : make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 s4 = in_row ? *(const float4*)(p.s + c4) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      v[i] = layer_norm4<KL>(v[i], g4, s4, inv, in_row);
    }
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) split4(v[i], pl[i]);
  stage();
  __syncthreads();

  // this lane's A operand rows: planes 0 and 1 from one LDS base, plane 2 from another (the
  // immediate offsets of LDS reads end at 64 KB)
  const bf16* arow = &P[0][(lane & 31) * kLdP + (lane >> 5) * 8];
  const bf16* arow2 = arow + 2 * ROWS * kLdP;
  f32x16 hi[TM], lo[TM];
  // hi/lo += the panel's rows x the weights streaming from cur (the stream goes on at next).
  // beside(ks) is work for the vector ALUs next to K step ks.
  auto multiply = [&](const char* cur, const char* next, auto&& beside) {
    bf16x8 a[2][TM][3];
    auto read_a = [&](bf16x8 (&d)[TM][3], int ks) {   // in the order of use
#pragma unroll
      for (int mi = 0; mi < TM; ++mi)
        d[mi][2] = *(const bf16x8*)(arow2 + mi * 32 * kLdP + ks * 16);
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
          d[mi][q] = *(const bf16x8*)(arow + q * (ROWS * kLdP) + mi * 32 * kLdP + ks * 16);
    };
    read_a(a[0], 0);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      asm volatile("" ::: "memory");   // one step's operands ahead, not a whole panel's
      const int s = ks % kDepth;
      if (ks + 1 < NKS) read_a(a[(ks + 1) & 1], ks + 1);
      // the small terms first; hi hi apart
      constexpr int ia[6] = {2, 0, 1, 1, 0, 0}, ib[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
      for (int t = 0; t < 6; ++t) {
#pragma unroll
        for (int mi = 0; mi < TM; ++mi) {
          f32x16& acc = t == 5 ? hi[mi] : lo[mi];
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              a[ks & 1][mi][ia[t]], __builtin_bit_cast(bf16x8, ring[s][ib[t]]), acc, 0, 0, 0);
        }
      }
      const char* src = (ks + kDepth < NKS ? cur + (ks + kDepth) * kStep
                                           : next + (ks + kDepth - NKS) * kStep);
#pragma unroll
      for (int q = 0; q < 3; ++q) ring[s][q] = *(const u32x4*)(src + q * 1024 + l16);
      beside(ks);
      // the next step's operand reads and the work beside spread over this step's products (left
      // alone, the compiler puts each read right before its product and waits for it)
#pragma unroll
      for (int t = 0; t < 3 * TM; ++t) {
        __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 1, 0);
        __builtin_amdgcn_sched_group_barrier(kSchedMfma, 2, 0);
        __builtin_amdgcn_sched_group_barrier(kSchedValu, 8, 0);
      }
      __builtin_amdgcn_sched_group_barrier(kSchedVmemRead, 3, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto zero = [&] {
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
      for (int r = 0; r < 16; ++r) hi[mi][r] = 0.f, lo[mi][r] = 0.f;
  };
  // hi = the finished sums
  auto finish = [&](int col) {
    const float bv = p.bias ? p.bias[col] : 0.f;
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
      for (int r = 0; r < 16; ++r) hi[mi][r] = (hi[mi][r] + lo[mi][r]) + bv;
  };
  // element (mi, r) of the accumulators: row 32 mi + 8 (r/4) + 4 (lane/32) + r%4, column col;
  // its address as a wave-uniform base and one 32-bit lane offset
  auto c_off = [&](int col) {
    uint32_t off = (uint32_t)((4 * (lane >> 5) * p.ldc + col) * 4);
    asm volatile("" : "+v"(off));
    return off;
  };
  auto c_at = [&](uint32_t off, int mi, int r) -> float* {
    char* row = (char*)(p.C + (m0 + mi * 32 + 8 * (r >> 2) + (r & 3)) * p.ldc);
    return (float*)(row + off);
  };
  if constexpr (EPI == EPI_RESID) {
    // one column block per wave at most; waves without one take part in the staging
    const int nb = nb0 + w, col = nb * 32 + (lane & 31);
    const bool on = nb < nb1;                       // wave-uniform
    if (!MULTI && !on) return;
    zero();
    const char* cur = wbase + nb * block_bytes;
    for (int panel = 0; panel < n_panels; ++panel, cur += NKS * kStep) {
      const bool more = panel + 1 < n_panels;
      if (MULTI && panel > 0) {
        __syncthreads();                            // the planes are consumed
        stage();
        __syncthreads();
      }
      if (MULTI) load(more ? panel + 1 : panel);
      // the next panel's rows are split beside the second half of the products
      auto split_next = [&](int ks) {
        if constexpr (MULTI) {
          if (ks >= NKS / 2 && ks - NKS / 2 < NI) split4(v[ks - NKS / 2], pl[ks - NKS / 2]);
        }
      };
      if (on) {
        multiply(cur, more ? cur + NKS * kStep : cur, split_next);
      } else {
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) split_next(ks);
      }
    }
    if (!on) return;
    finish(col);
    __builtin_amdgcn_sched_barrier(0);              // the sums first: half the registers
    const uint32_t off = c_off(col);
    float old[TM][16];
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
      for (int r = 0; r < 16; ++r) old[mi][r] = *c_at(off, mi, r);
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
      for (int r = 0; r < 16; ++r) *c_at(off, mi, r) = old[mi][r] + hi[mi][r];
  } else {
    for (int nb = nb0 + w; nb < nb1; nb += kNw) {
      const int col = nb * 32 + (lane & 31);
      const char* cur = wbase + nb * block_bytes;
      zero();
      multiply(cur, nb + kNw < nb1 ? cur + kNw * block_bytes : cur, [](int) {});
      finish(col);
      const uint32_t off = c_off(col);
#pragma unroll
      for (int mi = 0; mi < TM; ++mi)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int64_t row = m0 + mi * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
          const float o = EPI == EPI_GELU ? gelu_f32(hi[mi][r]) : hi[mi][r];
          if (SRC != SRC_EMBED_LN || row < p.m_store) *c_at(off, mi, r) = o;
        }
    }
  }
}

// One kernel name per class of product (the names of the general kernels), so that profiles
// separate them.
#define FMD_SPLIT_KERNEL(NAME)                                                               \
  template <int TM, int SRC, int EPI, int NKS, bool MULTI = false>                           \
  __global__ __launch_bounds__(kNt) __attribute__((amdgpu_waves_per_eu(2))) void NAME(       \
      SplitArgs p) {                                                                         \
    split_body<TM, SRC, EPI, NKS, MULTI>(p);                                                 \
  }
FMD_SPLIT_KERNEL(k_gemm_qkv)
FMD_SPLIT_KERNEL(k_gemm_proj)
FMD_SPLIT_KERNEL(k_gemm_qc)
FMD_SPLIT_KERNEL(k_gemm_up)
FMD_SPLIT_KERNEL(k_gemm_down)
FMD_SPLIT_KERNEL(k_gemm_kv)
#undef FMD_SPLIT_KERNEL

__global__ void k_pack_split(const float* __restrict__ W, int K, int N, u32x4* __restrict__ Wf) {
  const int nks = K / 16;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)(N / 32) * nks * 64) return;
  const int lane = (int)(e % 64);
  const int64_t f = e / 64;                          // fragment (nb, ks)
  const int ks = (int)(f % nks), nb = (int)(f / nks), n = nb * 32 + (lane & 31);
  bf16x8 v[3];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    float x[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = W[(int64_t)(ks * 16 + (lane >> 5) * 8 + 4 * h + j) * N + n];
    bf16x4 pl[3];
    split4(make_float4(x[0], x[1], x[2], x[3]), pl);
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j) v[q][4 * h + j] = pl[q][j];
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) Wf[(f * 3 + q) * 64 + lane] = __builtin_bit_cast(u32x4, v[q]);
}

// ---------------------------------------------------------------------------------------

bool split_supported(int d_model) { return d_model % 64 == 0 && d_model <= kPanel; }

size_t split_bytes(int64_t K, int64_t N) { return (size_t)(K * N) * 6; }

hipError_t launch_pack_split(hipStream_t st, const float* W, int K, int N, void* Wf) {
  if (K % 16 || N % 32) return hipErrorInvalidValue;
  const int64_t n = (int64_t)(N / 32) * (K / 16) * 64;
  hipLaunchKernelGGL(k_pack_split, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, W, K, N,
                     (u32x4*)Wf);
  return hipGetLastError();
}

namespace {
using SplitKernel = void (*)(SplitArgs);

template <int TM, int NKS>
SplitKernel split_kernel(int cls) {
  switch (cls) {
    case SPLIT_QKV: return k_gemm_qkv<TM, SRC_LN, EPI_STORE, NKS>;
    case SPLIT_QKV_EMBED: return k_gemm_qkv<TM, SRC_EMBED_LN, EPI_STORE, NKS>;
    case SPLIT_PROJ:
    case SPLIT_PROJ_CROSS: return k_gemm_proj<TM, SRC_ROWS, EPI_RESID, NKS>;
    case SPLIT_QC: return k_gemm_qc<TM, SRC_LN, EPI_STORE, NKS>;
    case SPLIT_UP: return k_gemm_up<TM, SRC_LN, EPI_GELU, NKS>;
    case SPLIT_DOWN: return k_gemm_down<TM, SRC_ROWS, EPI_RESID, kPanel / 16, true>;
    case SPLIT_KV: return k_gemm_kv<TM, SRC_EMBED_LN, EPI_STORE, NKS>;
    default: return nullptr;
  }
}

template <int TM>
SplitKernel split_kernel(int cls, int kp) {
  switch (kp) {
    case 64: return split_kernel<TM, 4>(cls);
    case 128: return split_kernel<TM, 8>(cls);
    case 192: return split_kernel<TM, 12>(cls);
    case 256: return split_kernel<TM, 16>(cls);
    default: return nullptr;
  }
}
}  // namespace

// Candidates of the autotuner (the results do not depend on the choice): 0: 64 rows per
// workgroup, which uses each weight fragment twice; 1: 32 rows; 2, 3: 32 rows with the passes of
// eight column blocks spread over two workgroups, and over one each. The rule where nothing is
// tuned: 64 rows once those tiles fill the 256 CUs, below that 32-row tiles and as many column
// parts as it takes.
bool split_tile(int cand, int64_t Mp, int N, int* rows, int* parts) {
  constexpr int64_t kCus = 256;
  const int passes = (N / 32 + kNw - 1) / kNw;
  if (cand < 0) {
    *rows = Mp / 64 >= kCus ? 64 : 32;
    *parts = 1;
    while (*parts < passes && Mp / *rows * *parts < kCus) ++*parts;
    return true;
  }
  *rows = cand == 0 ? 64 : 32;
  *parts = cand == 2 ? 2 : cand == 3 ? passes : 1;
  return cand < kSplitCands && (cand < 2 || passes > cand - 1);
}

hipError_t launch_split_gemm(hipStream_t st, int cls, int64_t Mp, SplitArgs p, int cand) {
  const int K = p.K, N = p.N;
  const bool ln = cls == SPLIT_QKV || cls == SPLIT_QC || cls == SPLIT_UP;
  const bool embed = cls == SPLIT_QKV_EMBED || cls == SPLIT_KV;
  if (Mp < 0 || Mp % kGemmBM || K % 64 || K <= 0 || N % 64 || N <= 0 || !p.A || !p.Wf || !p.C)
    return hipErrorInvalidValue;
  // several panels are whole ones, and only rows that are not normalised have them
  if (cls == SPLIT_DOWN ? K % kPanel != 0 : K > kPanel) return hipErrorInvalidValue;
  // residual products have at most eight column blocks
  if ((cls == SPLIT_DOWN || cls == SPLIT_PROJ || cls == SPLIT_PROJ_CROSS) && N > 32 * kNw)
    return hipErrorInvalidValue;
  if ((ln || embed) && (!p.g || !p.s)) return hipErrorInvalidValue;
  if (embed && (!p.Win || !p.base || p.lda < 9)) return hipErrorInvalidValue;
  if (!embed && p.lda % 4) return hipErrorInvalidValue;
  if (Mp == 0) return hipSuccess;
  int rows = 0, parts = 0;
  if (!split_tile(cand, Mp, N, &rows, &parts)) return hipErrorInvalidValue;
  const int n_blocks = N / 32, passes = (n_blocks + kNw - 1) / kNw;
  p.nb_per = (passes + parts - 1) / parts * kNw;
  const dim3 grid((unsigned)(Mp / rows), (unsigned)((n_blocks + p.nb_per - 1) / p.nb_per));
  const int kp = K < kPanel ? K : kPanel;
  SplitKernel k = rows == 64 ? split_kernel<2>(cls, kp) : split_kernel<1>(cls, kp);
  if (!k) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k, grid, dim3(kNt), 0, st, p);
  return hipGetLastError();
}

}  // namespace fmd
