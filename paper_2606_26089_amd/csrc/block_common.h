// Helpers of the fused BF16 block kernels shared by the throughput forms (block_bf16.hip) and
// the small-call forms (block_small.hip): operand layouts, row access, GELU, FP8 operands and
// the argument records of the chained tails.
#pragma once

#include "common.h"
#include "kernels.h"

namespace fmd {
namespace {

constexpr int kD = 256;              // model width
constexpr int kDh = 32;              // head width: wave w of a 256-wide slab = head w
constexpr int kWaves = 8;            // wave w owns columns [32w, 32w + 32) of a 256-wide slab
constexpr int kThreads = 64 * kWaves;
constexpr int kLdA = kD + 8;         // LDS pitch (bf16) of a 256-wide activation tile
constexpr int kKs = kD / 16;         // fragments along K = 256

__device__ __forceinline__ int acc_row(int mi, int r, int lane) {
  return mi * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
}

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// Global row access in the accumulator layout. Element (mi, r) of a lane sits at byte
// (32 mi + 8 (r/4) + r%4) * pitch + lane_off from the tile's first row, where
// lane_off = (4 (lane/32) * ld + col) * sizeof(elem). The row-group part is added to a
// wave-uniform base and r%4 becomes an immediate offset, so only one 32-bit per-lane
// offset stays live instead of one 64-bit address per element.
template <typename E, int LD>
struct RowIo {
  const char* base;     // wave-uniform: first row of the tile
  uint32_t lane_off;
  __device__ RowIo(const E* X, int64_t m0, int col, int lane)
      : base((const char*)(X + m0 * LD)),
        lane_off((uint32_t)((4 * (lane >> 5) * LD + col) * sizeof(E))) {
    // opaque to the compiler: the addresses are formed here, where they are used, and not
    // computed early and held live across the phases in between
    asm volatile("" : "+v"(lane_off));
  }
  __device__ __forceinline__ E* at(int mi, int r) const {
    const char* gb = base + (size_t)(mi * 32 + 8 * (r >> 2)) * LD * sizeof(E);
    return (E*)(gb + lane_off + (r & 3) * LD * sizeof(E));
  }
};

// Every row and tile transfer of these kernels is a non-temporal load or store: the rows
// stream through once, and kept in L2 they would evict the weight fragments that every
// workgroup re-reads.
//
// ROWS x 256 BF16 tile at rows m0.. of a head-major attention output [8 heads][Mp][32]
// (plane = Mp x 32 elements) into LDS (pitch kLdA, row-major): consecutive threads read
// consecutive 16-byte chunks of one head's rows.
template <int ROWS, int NT = kThreads>
__device__ __forceinline__ void tile_hm_to_lds(bf16* __restrict__ A, const bf16* __restrict__ S,
                                               int64_t plane, int64_t m0, int tid) {
  constexpr int kChunks = ROWS * kD / 8;                // 16-byte chunks
  constexpr int kPer = kChunks / NT;
  constexpr int kHeadChunks = ROWS * kDh / 8;           // chunks of one head's rows
  u32x4 v[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int idx = tid + i * NT, hd = idx / kHeadChunks, rem = idx % kHeadChunks;
    const u32x4* src = (const u32x4*)((const char*)(S + hd * plane + m0 * kDh) + (uint32_t)rem * 16);
    v[i] = __builtin_nontemporal_load(src);
  }
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int idx = tid + i * NT, hd = idx / kHeadChunks, rem = idx % kHeadChunks;
    *(u32x4*)(A + (rem / (kDh / 8)) * kLdA + hd * kDh + (rem % (kDh / 8)) * 8) = v[i];
  }
}

// Cross-lane data movement inside 16-lane rows (DPP controls).
constexpr int kDppXor1 = 0xB1;        // quad_perm [1,0,3,2]: lane i <- lane i ^ 1
constexpr int kDppXor2 = 0x4E;        // quad_perm [2,3,0,1]: lane i <- lane i ^ 2
constexpr int kDppHalfMirror = 0x141; // lane i <- lane 7 - i within each group of 8
constexpr int kDppRor8 = 0x128;       // lane i <- lane (i + 8) mod 16, i.e. i ^ 8

// GELU(z) = z/2 (1 + erf(z / sqrt 2)) with erf by Abramowitz & Stegun 7.1.27:
// erf(x) = 1 - (1 + a1 x + a2 x^2 + a3 x^3 + a4 x^4)^-4 for x >= 0, absolute error at most
// 5e-4, far below the BF16 rounding of the result (relative step 2^-8). Branch-free (a
// library erf branches on |x|), one hardware reciprocal and no exponential. The variable is
// u = z / sqrt(2 ln 2) (the callers fold the bias into it as bu = bias / sqrt(2 ln 2)), so
// x = |u| sqrt(ln 2), whose powers are folded into the coefficients b_k = a_k (ln 2)^(k/2);
// with h = sqrt(ln 2 / 2), GELU = h (u + |u| erf(x)). 10 vector instructions per value.
constexpr float kGeluU = 0.84932180028801904f;   // 1 / sqrt(2 ln 2)
__device__ __forceinline__ float gelu_as(float a, float bu) {
  constexpr float s = 0.83255461115769775f;   // sqrt(ln 2)
  constexpr float b1 = 0.278393f * s, b2 = 0.230389f * s * s, b3 = 0.000972f * s * s * s,
                  b4 = 0.078108f * s * s * s * s;
  constexpr float h = 0.5f / kGeluU;
  const float u = fmaf(a, kGeluU, bu);
  const float x = fabsf(u);
  float q = fmaf(b4, x, b3);
  q = fmaf(q, x, b2);
  q = fmaf(q, x, b1);
  q = fmaf(q, x, 1.0f);
  q = q * q;
  const float r = __builtin_amdgcn_rcpf(q * q);
  const float he = fmaf(-h, r, h);                  // h erf(|x|)
  return fmaf(x, he, u * h);
}

// sched_barrier mask: instructions of these kinds may be scheduled across it (VALU 0x2,
// SALU 0x4, LDS reads 0x100); vector-memory loads and MFMAs may not
constexpr int kKeepLoadsAndMfma = 0x2 | 0x4 | 0x100;

// Input embedding of block 0, formed in the QKV kernel instead of read from H, for a stage
// whose time is the same for every row: row r is temb + sum_k xs[r][k] W_xin[k] over the 9
// state features, in that order (the order of the embedding kernel, so the rows are the
// same), and is stored to H. Rows at or past T (padding) are zero. (Per-event times would
// need a time-embedding row per tile row; those calls keep the embedding kernel.)
struct EmbedRows {
  const float* xs;             // state rows, pitch kEmbLd floats, first 9 used
  int64_t T;
  const float* temb;           // [stages][256] time embeddings, b_xin included
  StageCtl* ctl;               // the current stage (null: row 0)
  const float* W;              // W_xin [9][256]
  float* H;                    // [Mp][256] output
};
constexpr int kEmbLd = 16;     // pitch of the ODE state rows
constexpr int kEmbF9 = 9;

// Which row tiles a launch covers: tile b of the grid is rows [ROWS t, ROWS t + ROWS) with
// t = tiles[b] when a map is given (the serving loop skips the tiles of gaps between
// requests), t = b otherwise. Mp is the padded row count of the call: the head-major planes
// hold Mp rows each, whatever tiles run.
struct RowMap {
  const int32_t* tiles;
  int64_t Mp;
  __device__ __forceinline__ int64_t first_row(int rows) const {
    return (int64_t)(tiles ? tiles[blockIdx.x] : (int32_t)blockIdx.x) * rows;
  }
};

// ---- FP8 (OCP e4m3) operands of the MLP's two projections (the FP8 precision form).
// The LayerNorm tile and the hidden chunks are FP8 bytes in LDS; W_up and W_dn are FP8
// fragments of the weights times a power of two per output column (so that the column's
// largest magnitude lies in (224, 448]) for the 32 x 32 x 64 matrix instruction: fragment
// (nb, ks) of lane l holds W[64 ks + 32 (l/32) + j][32 nb + l%32] s_col, j < 32, as 32 bytes,
// stored [N/32][K/64][64 lanes]. A operands from LDS take the same k order (row l%32, bytes
// 64 ks + 32 (l/32) ..), so products pair the same k on both sides. The up-projection output
// is scaled back by 1/s per hidden column before the GELU; the down-projection accumulates
// onto the residual rows multiplied by s per output column and divides by it afterwards,
// exact for powers of two. Accumulation, statistics, GELU and residual stay FP32.
typedef int i32x8 __attribute__((ext_vector_type(8)));

struct Mlp8 {
  const i32x8* up;      // W_up s_up fragments [1024/32][256/64][64]
  const i32x8* dn;      // W_dn s_dn fragments [256/32][1024/64][64]
  const float* up_inv;  // 1 / s_up per hidden column [1024]
  const float* dn_scale;   // s_dn per output column [256]
  const float* dn_inv;  // 1 / s_dn [256]
};

constexpr int kLdA8 = kD + 16;        // bytes per row of the FP8 LayerNorm tile
constexpr int kKs8 = kD / 64;         // 64-deep K steps over d

__device__ __forceinline__ f32x16 mfma_f8(i32x8 a, i32x8 b, f32x16 c) {
  // block scales 2^(127 - 127) = 1: plain FP8 x FP8 products
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 127, 0, 127);
}

// x rounded to the nearest e4m3 value (ties to even), as one byte
__device__ __forceinline__ uint32_t to_fp8(float x) {
  return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(x, x, 0, false) & 0xFFu;
}

// A operand of one 32-row block: row `row` of an FP8 tile (pitch ld bytes), K step ks
__device__ __forceinline__ i32x8 lds_frag8(const uint8_t* __restrict__ t, int ld, int row, int ks,
                                           int lane) {
  const uint8_t* p = t + row * ld + ks * 64 + (lane >> 5) * 32;
  const u32x4 lo = *(const u32x4*)p, hi = *(const u32x4*)(p + 16);
  i32x8 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    r[i] = (int)lo[i];
    r[4 + i] = (int)hi[i];
  }
  return r;
}

struct NextQkv {
  const float* g;        // LN1 gain and shift of the next block
  const float* s;
  const u32x4* Wf;       // its W_qkv fragments
  const float* bias;
  bf16* qkv;             // [3][8 heads][Mp][32]
};

// With HEAD (the last block), the kernel applies the output head to the final rows instead:
// LN_f, the 9-wide projection (FP32, per-wave partial sums over the wave's 64 columns by the
// transpose-reduction, then the 4 wave partials in wave order) and the ODE update of the
// state, as the separate head kernel does; the residual rows are then not stored.
struct NextHead {
  const float* g;        // LN_f gain and shift
  const float* s;
  const float* Wt;       // W_out transposed: row c = weights of output c (c < 9), 256 wide
  const float* b;
  OdeArgs ode;
};

enum MlpTail { kTailStats = 0, kTailQkv = 1, kTailHead = 2 };

struct MlpTailArgs {
  NextQkv nq;
  NextHead nh;
  Mlp8 f8;
};
inline MlpTailArgs mlp_tail_args(const FusedMlpArgs& a) {
  MlpTailArgs t{};
  if (a.qkv) t.nq = NextQkv{a.g1n, a.s1n, (const u32x4*)a.Wf_qkv_n, a.b_qkv_n, (bf16*)a.qkv};
  if (a.head) t.nh = NextHead{a.gf, a.sf, a.Wt_out, a.b_out, *a.head};
  if (a.fp8)
    t.f8 = Mlp8{(const i32x8*)a.fp8->up, (const i32x8*)a.fp8->dn, a.fp8->up_inv, a.fp8->dn_scale,
                a.fp8->dn_inv};
  return t;
}

}  // namespace

// Whether a set of MLP kernel arguments is complete (block_bf16.hip).
bool fused_mlp_args(const FusedMlpArgs& a);

}  // namespace fmd
