// Masked multi-head attention over ragged CSR events on gfx950 matrix cores.
//
// The general kernel (heads of 16 and 64; heads of 32 have their own below): each workgroup
// takes one (event, 64-query tile) work item for one head. Each of its four waves owns 16
// queries. Keys and values of the event stream through LDS in chunks of 64 keys, with an
// online (running max / running sum) softmax. Keys of other events are never touched. Slots
// past the end of the event are excluded by a select before the exponential, and their K and
// V rows are zero-filled in LDS, so garbage cannot reach the result.
//
// The scores are formed transposed, S^T = K Q^T, on 16 x 16 MFMA tiles. Lane l then
// holds query l%16 and keys 4(l/16) + r, so a query's statistics need only two
// cross-lane exchanges (xor 16, xor 32). Those registers are already the B operand of
// O^T = V^T P^T. The MFMA contracts over slot positions, and V^T is read from LDS with
// the same key-to-slot assignment.
//   FP32: v_mfma_f32_16x16x4_f32 (one k per lane; lane group g = l/16 holds k = g)
//   BF16: v_mfma_f32_16x16x32_bf16 (8 consecutive k per lane group), or 16x16x16 for dh 16
// Accumulator layout: lane l, register r holds row 4(l/16) + r, column l%16.
#include <algorithm>
#include <vector>

#include "common.h"
#include "kernels.h"

namespace fmd {

constexpr int KC = 64;   // keys per LDS chunk
constexpr int QT = 64;   // queries per workgroup (4 waves x 16)

template <typename T> struct AttnPad { static constexpr int v = 4; };
template <> struct AttnPad<bf16> { static constexpr int v = 8; };

template <typename T, int DH>
__device__ __forceinline__ void attention_body(
    const T* __restrict__ Q, int ldq, const T* __restrict__ Kp, const T* __restrict__ Vp,
    int ldkv, T* __restrict__ O, int ldo, const AttnItem* __restrict__ work,
    float scale_log2e) {
  constexpr bool BF = sizeof(T) == 2;
  constexpr int PAD = AttnPad<T>::v;
  constexpr int DB = DH / 16;                 // 16-wide output blocks along dh
  constexpr int CH = 16 / sizeof(T);          // elements per 16-byte chunk
  constexpr int CPR = DH / CH;                // chunks per K/V row
  __shared__ __attribute__((aligned(16))) T Ks[KC][DH + PAD];
  __shared__ __attribute__((aligned(16))) T Vt[DH][KC + PAD];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, j = lane & 15;
  const AttnItem wk = work[blockIdx.x];     // rows are those of the item's query tile
  const int h = blockIdx.y;
  const int64_t qs = wk.q0, ks = wk.k0;
  const int nq = wk.nq, nk = wk.nk;
  const int qbase = wave * 16;
  const bool wave_active = qbase < nq;
  const int qi = qbase + j;
  const bool qvalid = qi < nq;
  const T* qrow = Q + (qs + (qvalid ? qi : 0)) * ldq + h * DH;

  // Q fragment (B operand of S^T = K Q^T).
  constexpr int QN = BF ? (DH == 16 ? 4 : 8 * (DH / 32)) : DH / 4;
  float qf32[BF ? 1 : QN];
  bf16x8 qb[BF && DH >= 32 ? DH / 32 : 1];
  bf16x4 qb4;
  if constexpr (BF) {
    if constexpr (DH == 16) {
      qb4 = *(const bf16x4*)(qrow + 4 * g);
      if (!qvalid) for (int i = 0; i < 4; ++i) qb4[i] = (bf16)0.f;
    } else {
#pragma unroll
      for (int m = 0; m < DH / 32; ++m) {
        qb[m] = *(const bf16x8*)(qrow + 32 * m + 8 * g);
        if (!qvalid) for (int i = 0; i < 8; ++i) qb[m][i] = (bf16)0.f;
      }
    }
  } else {
#pragma unroll
    for (int m = 0; m < QN; ++m) qf32[m] = qvalid ? to_f32(qrow[g * QN + m]) : 0.f;
  }

  float m_run = -INFINITY, l_run = 0.f;
  f32x4 o[DB];
#pragma unroll
  for (int b = 0; b < DB; ++b) o[b] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int c0 = 0; c0 < nk; c0 += KC) {
    // stage K rows and V^T columns of keys c0 .. c0 + 63
    for (int idx = tid; idx < KC * CPR; idx += 256) {
      const int row = idx / CPR, ch = idx % CPR;
      u32x4 kv = {0u, 0u, 0u, 0u}, vv = {0u, 0u, 0u, 0u};
      if (c0 + row < nk) {
        const int64_t gr = (ks + c0 + row) * ldkv + h * DH + ch * CH;
        kv = *(const u32x4*)(Kp + gr);
        vv = *(const u32x4*)(Vp + gr);
      }
      *(u32x4*)&Ks[row][ch * CH] = kv;
      const T* vp = (const T*)&vv;
#pragma unroll
      for (int i = 0; i < CH; ++i) Vt[ch * CH + i][row] = vp[i];
    }
    __syncthreads();
    if (wave_active) {
      f32x4 s[4];
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        s[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
        const T* krow = &Ks[kb * 16 + j][0];
        if constexpr (BF) {
          if constexpr (DH == 16) {
            const bf16x4 ka = *(const bf16x4*)(krow + 4 * g);
            s[kb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ka, qb4, s[kb], 0, 0, 0);
          } else {
#pragma unroll
            for (int m = 0; m < DH / 32; ++m) {
              const bf16x8 ka = *(const bf16x8*)(krow + 32 * m + 8 * g);
              s[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, qb[m], s[kb], 0, 0, 0);
            }
          }
        } else {
#pragma unroll
          for (int m = 0; m < QN; ++m)
            s[kb] = __builtin_amdgcn_mfma_f32_16x16x4f32(to_f32(krow[g * QN + m]), qf32[m],
                                                         s[kb], 0, 0, 0);
        }
      }
      float cmax = -INFINITY;
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int key = c0 + kb * 16 + 4 * g + r;
          const float v = key < nk ? s[kb][r] * scale_log2e : -INFINITY;
          s[kb][r] = v;
          cmax = fmaxf(cmax, v);
        }
      cmax = fmaxf(cmax, __shfl_xor(cmax, 16, kWave));
      cmax = fmaxf(cmax, __shfl_xor(cmax, 32, kWave));
      const float m_new = fmaxf(m_run, cmax);      // finite: key c0 < nk is in this chunk
      const float alpha = exp2f(m_run - m_new);
      l_run *= alpha;
#pragma unroll
      for (int b = 0; b < DB; ++b) o[b] *= alpha;
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float p = exp2f(s[kb][r] - m_new);
          s[kb][r] = p;
          l_run += p;
        }
      m_run = m_new;
      // O^T += V^T P^T
      if constexpr (BF) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          bf16x8 pb;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            pb[r] = (bf16)s[2 * c][r];
            pb[4 + r] = (bf16)s[2 * c + 1][r];
          }
#pragma unroll
          for (int b = 0; b < DB; ++b) {
            const T* vrow = &Vt[b * 16 + j][0];
            const bf16x4 lo = *(const bf16x4*)(vrow + 32 * c + 4 * g);
            const bf16x4 hi = *(const bf16x4*)(vrow + 32 * c + 16 + 4 * g);
            bf16x8 va;
#pragma unroll
            for (int r = 0; r < 4; ++r) { va[r] = lo[r]; va[4 + r] = hi[r]; }
            o[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, pb, o[b], 0, 0, 0);
          }
        }
      } else {
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
#pragma unroll
          for (int b = 0; b < DB; ++b) {
            const float4 va = *(const float4*)&Vt[b * 16 + j][kb * 16 + 4 * g];
            o[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(va.x, s[kb][0], o[b], 0, 0, 0);
            o[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(va.y, s[kb][1], o[b], 0, 0, 0);
            o[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(va.z, s[kb][2], o[b], 0, 0, 0);
            o[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(va.w, s[kb][3], o[b], 0, 0, 0);
          }
        }
      }
    }
    __syncthreads();
  }

  if (wave_active) {
    float l = l_run + __shfl_xor(l_run, 16, kWave);
    l += __shfl_xor(l, 32, kWave);
    const float inv = 1.0f / l;
    if (qvalid) {
      T* orow = O + (qs + qi) * ldo + h * DH;
#pragma unroll
      for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) orow[b * 16 + 4 * g + r] = from_f32<T>(o[b][r] * inv);
    }
  }
}

// Separate kernel names for self- and cross-attention so that profiles separate them.
#define FMD_ATTN_KERNEL(NAME)                                                                 \
  template <typename T, int DH>                                                               \
  __global__ __launch_bounds__(256) void NAME(                                                \
      const T* __restrict__ Q, int ldq, const T* __restrict__ K, const T* __restrict__ V,     \
      int ldkv, T* __restrict__ O, int ldo, const AttnItem* __restrict__ work, float sl2e) {  \
    attention_body<T, DH>(Q, ldq, K, V, ldkv, O, ldo, work, sl2e);                            \
  }
FMD_ATTN_KERNEL(k_attn_self)
FMD_ATTN_KERNEL(k_attn_cross)
#undef FMD_ATTN_KERNEL

// ---------------------------------------------------------------------------------------
// BF16 with heads of 32: the same work split as above (one head of one 64-query tile per
// workgroup, four waves of 16 queries), tuned for gfx950.
//  - Chunks of 128 keys: most events fit in one, so the load -> barrier -> compute round
//    trip is paid once. K rows are staged by waves 2-3 and V by waves 0-1, 4 loads each.
//    A last chunk of at most 96 keys is staged and computed for its first 32, 64 or 96 keys
//    only (a straight-line form for each, after the loop over full chunks).
//  - One-dimensional grid over (work item, head), heads fastest: the workgroups that read
//    the two halves of a K/V cache line run together, so the line is fetched once. (The
//    work list is sorted longest event first; dealing contiguous ranges of it to the XCDs
//    would load one XCD with all the long events.)
//  - V is staged transposed with packed 8-byte LDS stores (no two lanes write the same
//    dword) and with a key permutation inside each 32-key group (key 16 hi + 4 g + r at
//    position 8 g + 4 hi + r): the eight keys lane group g feeds to one MFMA are adjacent,
//    so each V^T operand is one 16-byte LDS read.
//  - The softmax runs on unscaled scores: one multiply-add forms the exp2 argument
//    (s - max) * scale, and the hardware exp2 is used (arguments <= 0). The row sums of P
//    come from the P V product itself, through a third 16-row block of V^T whose first row
//    is the key validity. Keys past the event end repeat its last key (clamped reads) and
//    have zero V and validity, so there is no per-score masking.
namespace {
constexpr int kH32 = 32;
constexpr int kKc2 = 128;           // keys per chunk
constexpr int kSchedMfma = 0x008;   // sched_group_barrier instruction classes: MFMA
constexpr int kSchedDsRead = 0x100; // LDS read
constexpr int kLdK32 = kH32 + 8;    // Ks pitch (bf16)
constexpr int kLdV32 = kKc2 + 8;    // Vt pitch (bf16)

__device__ __forceinline__ int vt_pos(int k) {
  const int grp = k >> 5, hi = (k >> 4) & 1, g = (k >> 2) & 3, r = k & 3;
  return grp * 32 + 8 * g + 4 * hi + r;
}
}  // namespace

// One staged chunk of KB key blocks of 16 for this wave's query tiles: the scores
// S^T = K Q^T, the online-softmax update of the running max and the output, and
// O^T += V^T P^T with the row sums of P from the validity row of V^T.
template <int TPW, int KB>
__device__ __forceinline__ void attn32_chunk(const bf16* __restrict__ Ks,
                                             const bf16* __restrict__ Vt,
                                             const bf16x8 (&qf)[TPW], float (&m_run)[TPW],
                                             f32x4 (&o)[TPW][3], int nq, int wave, int g, int j,
                                             float sl2e) {
  auto qbase = [&](int t) { return (t * 4 + wave) * 16; };
  // compiler-only barrier: the LDS reads (and so the products) of the forms of this
  // function are not merged and hoisted above the branches between them
  asm volatile("" ::: "memory");
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    if (qbase(t) >= nq) continue;   // wave-uniform
    // all KB key blocks, also past the event end: no branches, and the zero accumulator
    // is an inline constant
    f32x4 s[KB];
    {
      bf16x8 kf[KB];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) kf[kb] = *(const bf16x8*)&Ks[(kb * 16 + j) * kLdK32 + 8 * g];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
        s[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kb], qf[t], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      // the K operand reads kept two ahead of their products (left alone, the compiler reads
      // each one right before its product into the same registers and waits for it)
      __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 2, 0);
#pragma unroll
      for (int i = 0; i < KB - 2; ++i) {
        __builtin_amdgcn_sched_group_barrier(kSchedMfma, 1, 0);
        __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(kSchedMfma, 2, 0);
    }
    float cmax = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r) cmax = fmaxf(cmax, s[kb][r]);
    {   // max over lanes l, l ^ 16, then l, l ^ 32: a row swap and a half swap of the
        // register with itself, no LDS round trip (max is exact)
      const auto r16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(cmax),
                                                        __float_as_uint(cmax), false, false);
      cmax = fmaxf(__uint_as_float(r16[0]), __uint_as_float(r16[1]));
      const auto r32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(cmax),
                                                        __float_as_uint(cmax), false, false);
      cmax = fmaxf(__uint_as_float(r32[0]), __uint_as_float(r32[1]));
    }
    const float m_new = fmaxf(m_run[t], cmax);    // finite: key c0 < nk is in this chunk
    const float alpha = __builtin_amdgcn_exp2f((m_run[t] - m_new) * sl2e);
#pragma unroll
    for (int db = 0; db < 3; ++db) o[t][db] *= alpha;
    const float mb = -m_new * sl2e;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r) s[kb][r] = __builtin_amdgcn_exp2f(fmaf(s[kb][r], sl2e, mb));
    m_run[t] = m_new;
#pragma unroll
    for (int c = 0; c < KB / 2; ++c) {
      bf16x8 pb;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        pb[r] = (bf16)s[2 * c][r];
        pb[4 + r] = (bf16)s[2 * c + 1][r];
      }
#pragma unroll
      for (int db = 0; db < 2; ++db) {
        const bf16x8 vf = *(const bf16x8*)&Vt[(db * 16 + j) * kLdV32 + 32 * c + 8 * g];
        o[t][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pb, o[t][db], 0, 0, 0);
      }
      const bf16x8 vld = *(const bf16x8*)&Vt[(kH32 + j) * kLdV32 + 32 * c + 8 * g];
      o[t][2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vld, pb, o[t][2], 0, 0, 0);
    }
  }
}

// Stages keys c0 .. c0 + 16 KB - 1 of the event into Ks and V^T.
template <int KB>
__device__ __forceinline__ void attn32_stage(bf16* __restrict__ Ks, bf16* __restrict__ Vt,
                                             const bf16* __restrict__ Kp,
                                             const bf16* __restrict__ Vp, int ldkv, int64_t hskv,
                                             int64_t ks0, int c0, int nk, int h, int tid,
                                             int wave) {
  // Keys past the event end are read clamped to its last key: their scores repeat a real
  // score (the running max is unchanged), and their V rows and validity are zero, so they
  // add nothing to P V or to the row sums. No per-score masking is needed.
  const int lim = nk - 1 - c0;
  if (wave >= 2) {   // K: 16 KB keys x 4 chunks of 16 bytes
    const char* kc = (const char*)(Kp + (ks0 + c0) * ldkv + h * hskv);
    const int t2 = tid - 128;
    u32x4 v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int idx = t2 + i * 128, row = idx >> 2, ch = idx & 3;
      if (i < KB / 2) v[i] = *(const u32x4*)(kc + (uint32_t)((min(row, lim) * ldkv + ch * 8) * 2));
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int idx = t2 + i * 128, row = idx >> 2, ch = idx & 3;
      if (i < KB / 2) *(u32x4*)&Ks[row * kLdK32 + ch * 8] = v[i];
    }
  } else if ((tid & 31) < 4 * KB) {   // V^T: thread = (4 consecutive keys, 8 dims)
    const char* vc = (const char*)(Vp + (ks0 + c0) * ldkv + h * hskv);
    const int kg = tid & 31, dg = tid >> 5;
    u32x4 v[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int key = kg * 4 + r;
      v[r] = *(const u32x4*)(vc + (uint32_t)((min(key, lim) * ldkv + dg * 8) * 2));
      if (key > lim) v[r] = u32x4{0u, 0u, 0u, 0u};
    }
    const int pos = vt_pos(kg * 4);
    if (dg == 0) {
      bf16x4 valid;
#pragma unroll
      for (int r = 0; r < 4; ++r) valid[r] = (bf16)(kg * 4 + r <= lim ? 1.f : 0.f);
      *(bf16x4*)&Vt[kH32 * kLdV32 + pos] = valid;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      bf16x4 w4;
#pragma unroll
      for (int r = 0; r < 4; ++r) w4[r] = __builtin_bit_cast(bf16x8, v[r])[i];
      *(bf16x4*)&Vt[(dg * 8 + i) * kLdV32 + pos] = w4;
    }
  }
}

// Few rows leave most CUs idle, and the weights of all blocks (11 MB) do not stay in an XCD's 4 MB
// of L2 from one evaluation to the next: the kernels after this one would stream them from the
// last-level cache, an MLP launch 2 us longer than from L2 (105 rows: 20.8 -> 18.7 us). Extra
// workgroups of the launch read one word of every 128-byte line, eight lines a thread in flight;
// workgroup b runs on XCD b % 8, so each part of the range is read once per XCD.
constexpr uint32_t kTouchPart = 256 * 8 * 128;   // bytes per workgroup
__device__ __forceinline__ void touch_l2(const L2Touch& t, int tid) {
  const char* p = (const char*)t.p;
  const uint32_t off = (blockIdx.x - t.first) / kAttnBins * kTouchPart + tid * 128;
  uint32_t x = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) x ^= *(const uint32_t*)(p + min(off + i * 256 * 128, t.bytes - 4));
  asm volatile("" ::"v"(x));
}

template <int TPW>
__device__ __forceinline__ void attention32_body(
    const bf16* __restrict__ Q, int ldq, int64_t hsq, const bf16* __restrict__ Kp,
    const bf16* __restrict__ Vp, int ldkv, int64_t hskv, bf16* __restrict__ O, int ldo,
    int64_t hso, const AttnItem* __restrict__ work, const AttnBins& bins, int n_heads, float sl2e) {
  __shared__ __attribute__((aligned(16))) bf16 Ks[kKc2 * kLdK32];
  // V^T rows 0-31; row 32 = key validity (1 for a key of the event, 0 past its end), rows
  // 33-47 = 0: the A operand of the row-sum block of P V
  __shared__ __attribute__((aligned(16))) bf16 Vt[(kH32 + 16) * kLdV32];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, j = lane & 15;
  for (int i = tid; i < 15 * kLdV32; i += 256) Vt[(kH32 + 1) * kLdV32 + i] = (bf16)0.f;
  // workgroup b: bin b % kAttnBins (so one XCD), unit k = b / kAttnBins of that bin
  const int bin = blockIdx.x % kAttnBins, k = blockIdx.x / kAttnBins;
  const int item = k / n_heads;
  if (item >= bins.len[bin]) return;     // the bin is shorter than the longest one
  // the item carries its rows: no dependent loads of event offsets before the data loads
  const AttnItem wk = work[bins.start[bin] + item];
  const int h = k % n_heads;
  const int64_t qs0 = wk.q0, ks0 = wk.k0;
  const int nq = wk.nq, nk = wk.nk;
  // query tile t of this wave (16 queries): tiles are dealt to the waves round-robin
  auto qbase = [&](int t) { return (t * 4 + wave) * 16; };

  bf16x8 qf[TPW];
  float m_run[TPW];
  // o[t][0], o[t][1]: output dims 0-15, 16-31; o[t][2] row 0 (lanes 0-15, register 0): sum of P
  f32x4 o[TPW][3];
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int qi = qbase(t) + j;
    const char* qc = (const char*)(Q + qs0 * ldq + h * hsq);
    u32x4 v = *(const u32x4*)(qc + (uint32_t)((min(qi, nq - 1) * ldq + 8 * g) * 2));
    if (qi >= nq) v = u32x4{0u, 0u, 0u, 0u};
    qf[t] = __builtin_bit_cast(bf16x8, v);
    m_run[t] = -INFINITY;
#pragma unroll
    for (int db = 0; db < 3; ++db) o[t][db] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // A last chunk of at most 96 keys is staged and computed for its first 32, 64 or 96 keys
  // only: the rest are all past the event end (their scores repeat a real score, their
  // P V and row-sum terms are exact zeros), so the results are the same.
  const int last = (nk - 1) & (kKc2 - 1);           // last key's position in its chunk
  const int nfull = last < 96 ? nk - 1 - last : nk;  // keys before the shortened last chunk
  for (int c0 = 0; c0 < nfull; c0 += kKc2) {
    attn32_stage<8>(Ks, Vt, Kp, Vp, ldkv, hskv, ks0, c0, nk, h, tid, wave);
    __syncthreads();
    attn32_chunk<TPW, 8>(Ks, Vt, qf, m_run, o, nq, wave, g, j, sl2e);
    __syncthreads();
  }
  const int rest = nk - nfull;   // 0 .. 96, wave-uniform
  if (rest > 64) {
    attn32_stage<6>(Ks, Vt, Kp, Vp, ldkv, hskv, ks0, nfull, nk, h, tid, wave);
    __syncthreads();
    attn32_chunk<TPW, 6>(Ks, Vt, qf, m_run, o, nq, wave, g, j, sl2e);
  } else if (rest > 32) {
    attn32_stage<4>(Ks, Vt, Kp, Vp, ldkv, hskv, ks0, nfull, nk, h, tid, wave);
    __syncthreads();
    attn32_chunk<TPW, 4>(Ks, Vt, qf, m_run, o, nq, wave, g, j, sl2e);
  } else if (rest > 0) {
    attn32_stage<2>(Ks, Vt, Kp, Vp, ldkv, hskv, ks0, nfull, nk, h, tid, wave);
    __syncthreads();
    attn32_chunk<TPW, 2>(Ks, Vt, qf, m_run, o, nq, wave, g, j, sl2e);
  }

#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int qi = qbase(t) + j;
    if (qbase(t) >= nq) continue;
    // row 0 of the row-sum block sits in register 0 of lanes 0-15 (query j)
    const float l = __shfl(o[t][2][0], j, kWave);
    const float inv = 1.0f / l;
    if (qi < nq) {
      bf16* orow = O + (qs0 + qi) * ldo + h * hso;
#pragma unroll
      for (int db = 0; db < 2; ++db) {
        bf16x4 w4;
#pragma unroll
        for (int r = 0; r < 4; ++r) w4[r] = (bf16)(o[t][db][r] * inv);
        *(bf16x4*)(orow + db * 16 + 4 * g) = w4;
      }
    }
  }
}

template <int TPW>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_attn32_self(
    const bf16* __restrict__ Q, int ldq, int64_t hsq, const bf16* __restrict__ K,
    const bf16* __restrict__ V, int ldkv, int64_t hskv, bf16* __restrict__ O, int ldo,
    int64_t hso, const AttnItem* __restrict__ work, AttnBins bins, int n_heads, float sl2e,
    L2Touch touch) {
  if (blockIdx.x >= touch.first) return touch_l2(touch, threadIdx.x);
  attention32_body<TPW>(Q, ldq, hsq, K, V, ldkv, hskv, O, ldo, hso, work, bins, n_heads, sl2e);
}
template <int TPW>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_attn32_cross(
    const bf16* __restrict__ Q, int ldq, int64_t hsq, const bf16* __restrict__ K,
    const bf16* __restrict__ V, int ldkv, int64_t hskv, bf16* __restrict__ O, int ldo,
    int64_t hso, const AttnItem* __restrict__ work, AttnBins bins, int n_heads, float sl2e,
    L2Touch touch) {
  if (blockIdx.x >= touch.first) return touch_l2(touch, threadIdx.x);
  attention32_body<TPW>(Q, ldq, hsq, K, V, ldkv, hskv, O, ldo, hso, work, bins, n_heads, sl2e);
}


// ---------------------------------------------------------------------------------------
// FP32 with heads of 32: the split of k_attn32 (one head of one work item per workgroup, 16-query
// tiles dealt to four waves, XCD bins) with every product on the BF16 matrix cores as in the
// split GEMMs: Q, K, V and the probabilities as three BF16 parts each, the six partial products
// down to 2^-16 of the product in FP32 accumulators (96 instructions of 16 cycles for 16 queries
// and 128 keys, where the FP32 instruction takes 128 of 32). Row sums stay FP32 sums of the
// unsplit probabilities.
//  - Chunks of 64 keys (29 KB of LDS, five workgroups per CU), the next chunk's rows in registers
//    while the current one is computed. K is split as it is staged, 8 dims a thread; V is staged
//    transposed in the key order of vt_pos, four keys a store.
//  - Only a chunk that the event ends in is masked; one of at most 32 keys is computed for 32.
// Bound: staging, products and softmax of a chunk in turn per workgroup, as in k_attn32; 448,552
// rows: 1050 -> 650 us a launch (2.8 TB/s), 14,276 rows: 46 -> 26 us, against the FP32 matrix
// instruction with 64-query items.
namespace {
constexpr int kKcF = 64;              // keys per chunk
constexpr int kLdKF = kH32 + 8;       // Ks pitch (bf16)
constexpr int kLdVF = kKcF + 8;       // Vt pitch (bf16)

// x = hi + mid + lo for eight values (hi truncated, mid and lo rounded to nearest)
__device__ __forceinline__ void split8(const float (&x)[8], bf16x8 (&p)[3]) {
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint32_t hb = __float_as_uint(x[i]) & 0xffff0000u;
    const float r = x[i] - __uint_as_float(hb);
    const bf16 mid = (bf16)r;
    p[0][i] = __builtin_bit_cast(bf16, (uint16_t)(hb >> 16));
    p[1][i] = mid;
    p[2][i] = (bf16)(r - (float)mid);
  }
}

// acc += A B over 32 k, the small partial products first
__device__ __forceinline__ f32x4 mfma_split(const bf16x8 (&a)[3], const bf16x8 (&b)[3], f32x4 acc) {
  constexpr int ia[6] = {2, 0, 1, 1, 0, 0}, ib[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
  for (int t = 0; t < 6; ++t)
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ia[t]], b[ib[t]], acc, 0, 0, 0);
  return acc;
}

struct AttnLdsF {
  bf16 Ks[3][kKcF * kLdKF];
  bf16 Vt[3][kH32 * kLdVF];
};
}  // namespace

// One staged chunk of KB key blocks of 16, `rest` of its keys in the event.
template <int TPW, int KB>
__device__ __forceinline__ void attn32f_chunk(const AttnLdsF& L, const bf16x8 (&qf)[TPW][3],
                                              float (&m_run)[TPW], float (&l_run)[TPW],
                                              f32x4 (&o)[TPW][2], int nq, int rest, int wave, int g,
                                              int j, float sl2e) {
  asm volatile("" ::: "memory");   // the forms' LDS reads are not merged above their branches
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    if ((t * 4 + wave) * 16 >= nq) continue;   // wave-uniform
    f32x4 s[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      bf16x8 kf[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) kf[q] = *(const bf16x8*)&L.Ks[q][(kb * 16 + j) * kLdKF + 8 * g];
      s[kb] = mfma_split(kf, qf[t], f32x4{0.f, 0.f, 0.f, 0.f});
    }
    if (rest < 16 * KB) {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (kb * 16 + 4 * g + r >= rest) s[kb][r] = -INFINITY;
    }
    float cmax = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r) cmax = fmaxf(cmax, s[kb][r]);
    {
      const auto r16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(cmax),
                                                        __float_as_uint(cmax), false, false);
      cmax = fmaxf(__uint_as_float(r16[0]), __uint_as_float(r16[1]));
      const auto r32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(cmax),
                                                        __float_as_uint(cmax), false, false);
      cmax = fmaxf(__uint_as_float(r32[0]), __uint_as_float(r32[1]));
    }
    const float m_new = fmaxf(m_run[t], cmax);    // finite: the chunk holds a key of the event
    const float alpha = __builtin_amdgcn_exp2f((m_run[t] - m_new) * sl2e);
    m_run[t] = m_new;
    const float mb = -m_new * sl2e;
    float l = l_run[t] * alpha;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[kb][r] = __builtin_amdgcn_exp2f(fmaf(s[kb][r], sl2e, mb));
        l += s[kb][r];
      }
    l_run[t] = l;
#pragma unroll
    for (int db = 0; db < 2; ++db) o[t][db] *= alpha;
#pragma unroll
    for (int c = 0; c < KB / 2; ++c) {
      float pv[8];
#pragma unroll
      for (int r = 0; r < 4; ++r) pv[r] = s[2 * c][r], pv[4 + r] = s[2 * c + 1][r];
      bf16x8 pf[3];
      split8(pv, pf);
#pragma unroll
      for (int db = 0; db < 2; ++db) {
        bf16x8 vf[3];
#pragma unroll
        for (int q = 0; q < 3; ++q)
          vf[q] = *(const bf16x8*)&L.Vt[q][(db * 16 + j) * kLdVF + 32 * c + 8 * g];
        o[t][db] = mfma_split(vf, pf, o[t][db]);
      }
    }
  }
}

template <int TPW>
__device__ __forceinline__ void attention32f_body(
    const float* __restrict__ Q, int ldq, int64_t hsq, const float* __restrict__ Kp,
    const float* __restrict__ Vp, int ldkv, int64_t hskv, float* __restrict__ O, int ldo,
    int64_t hso, const AttnItem* __restrict__ work, const AttnBins& bins, int n_heads, float sl2e) {
  __shared__ __attribute__((aligned(16))) AttnLdsF L;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, j = lane & 15;
  const int bin = blockIdx.x % kAttnBins, k = blockIdx.x / kAttnBins;
  const int item = k / n_heads;
  if (item >= bins.len[bin]) return;     // the bin is shorter than the longest one
  const AttnItem wk = work[bins.start[bin] + item];
  const int h = k % n_heads;
  const int nq = wk.nq, nk = wk.nk;
  const float* kc = Kp + (int64_t)wk.k0 * ldkv + h * hskv;
  const float* vc = Vp + (int64_t)wk.k0 * ldkv + h * hskv;

  // staging: thread = (key, 8 dims) of K and (4 consecutive keys, 2 dims) of V; keys past the
  // event end read its last key (K: masked scores) or are zero (V)
  const int kkey = tid >> 2, kch = tid & 3, vkg = tid >> 4, vdg = tid & 15;
  float4 rk[2];
  float2 rv[4];
  auto load = [&](int c0) {
    const int lim = nk - 1 - c0;
    const float* kr = kc + (int64_t)(c0 + min(kkey, lim)) * ldkv + 8 * kch;
    rk[0] = *(const float4*)kr;
    rk[1] = *(const float4*)(kr + 4);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int key = 4 * vkg + r;
      rv[r] = *(const float2*)(vc + (int64_t)(c0 + min(key, lim)) * ldkv + 2 * vdg);
      if (key > lim) rv[r] = make_float2(0.f, 0.f);
    }
  };
  auto stage = [&]() {
    const float kx[8] = {rk[0].x, rk[0].y, rk[0].z, rk[0].w, rk[1].x, rk[1].y, rk[1].z, rk[1].w};
    const float vx[8] = {rv[0].x, rv[1].x, rv[2].x, rv[3].x, rv[0].y, rv[1].y, rv[2].y, rv[3].y};
    bf16x8 kp[3], vp[3];
    split8(kx, kp);
    split8(vx, vp);
    const int pos = vt_pos(4 * vkg);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      *(bf16x8*)&L.Ks[q][kkey * kLdKF + 8 * kch] = kp[q];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        bf16x4 w4;
#pragma unroll
        for (int r = 0; r < 4; ++r) w4[r] = vp[q][4 * i + r];
        *(bf16x4*)&L.Vt[q][(2 * vdg + i) * kLdVF + pos] = w4;
      }
    }
  };

  load(0);
  bf16x8 qf[TPW][3];
  float m_run[TPW], l_run[TPW];
  f32x4 o[TPW][2];
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int qi = (t * 4 + wave) * 16 + j;
    const float* qr = Q + (int64_t)(wk.q0 + min(qi, nq - 1)) * ldq + h * hsq + 8 * g;
    const float4 a = *(const float4*)qr, b = *(const float4*)(qr + 4);
    const float qx[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    split8(qx, qf[t]);
    m_run[t] = -INFINITY;
    l_run[t] = 0.f;
#pragma unroll
    for (int db = 0; db < 2; ++db) o[t][db] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  for (int c0 = 0; c0 < nk; c0 += kKcF) {
    if (c0) __syncthreads();             // the chunk before is consumed
    stage();
    if (c0 + kKcF < nk) load(c0 + kKcF);
    __syncthreads();
    const int rest = nk - c0;
    if (rest > 32)
      attn32f_chunk<TPW, 4>(L, qf, m_run, l_run, o, nq, rest, wave, g, j, sl2e);
    else
      attn32f_chunk<TPW, 2>(L, qf, m_run, l_run, o, nq, rest, wave, g, j, sl2e);
  }
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int qi = (t * 4 + wave) * 16 + j;
    if ((t * 4 + wave) * 16 >= nq) continue;
    float l = l_run[t] + __shfl_xor(l_run[t], 16, kWave);
    l += __shfl_xor(l, 32, kWave);
    const float inv = 1.0f / l;
    if (qi < nq) {
      float* orow = O + (int64_t)(wk.q0 + qi) * ldo + h * hso + 4 * g;
#pragma unroll
      for (int db = 0; db < 2; ++db)
        *(float4*)(orow + db * 16) = make_float4(o[t][db][0] * inv, o[t][db][1] * inv,
                                                 o[t][db][2] * inv, o[t][db][3] * inv);
    }
  }
}

#define FMD_ATTN32F_KERNEL(NAME)                                                               \
  template <int TPW>                                                                           \
  __global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void NAME(         \
      const float* __restrict__ Q, int ldq, int64_t hsq, const float* __restrict__ K,          \
      const float* __restrict__ V, int ldkv, int64_t hskv, float* __restrict__ O, int ldo,     \
      int64_t hso, const AttnItem* __restrict__ work, AttnBins bins, int n_heads, float sl2e) { \
    attention32f_body<TPW>(Q, ldq, hsq, K, V, ldkv, hskv, O, ldo, hso, work, bins, n_heads,    \
                           sl2e);                                                              \
  }
FMD_ATTN32F_KERNEL(k_attn_self)
FMD_ATTN32F_KERNEL(k_attn_cross)
#undef FMD_ATTN32F_KERNEL

template <typename T, int DH>
static hipError_t go_attn(bool cross, dim3 grid, hipStream_t st, const T* Q, int ldq,
                          const T* K, const T* V, int ldkv, T* O, int ldo,
                          const AttnItem* work, float sl2e) {
  if (cross)
    hipLaunchKernelGGL((k_attn_cross<T, DH>), grid, dim3(256), 0, st, Q, ldq, K, V, ldkv, O, ldo,
                       work, sl2e);
  else
    hipLaunchKernelGGL((k_attn_self<T, DH>), grid, dim3(256), 0, st, Q, ldq, K, V, ldkv, O, ldo,
                       work, sl2e);
  return hipGetLastError();
}

namespace {
// The builder over accessors: queries of event k at q_off[ids[k]], nq(k) rows; its keys at
// k0(k), nk(k) rows.
template <typename Nq, typename K0, typename Nk>
int64_t build_work(const int64_t* q_off, const int64_t* ids, int64_t n, int qt, int deal, Nq nq,
                   K0 k0, Nk nk, AttnItem* items, AttnBins* bins) {
  // longest-processing-time assignment of whole events to bins; cost = query tiles x keys. With
  // `deal` heads, the tiles of an event of more than two workgroups for each CU of an XCD that holds
  // more than a quarter of a bin's fair share go to the least loaded bin one by one.
  std::vector<int64_t> order;
  order.reserve((size_t)n);
  for (int64_t k = 0; k < n; ++k) {
    if (nq(k) <= 0) continue;
    if (q_off[ids[k]] + nq(k) > INT32_MAX || k0(k) + nk(k) > INT32_MAX) return -1;
    order.push_back(k);
  }
  auto tiles = [&](int64_t k) { return (nq(k) + qt - 1) / qt; };
  auto cost = [&](int64_t k) { return tiles(k) * nk(k); };
  std::stable_sort(order.begin(), order.end(), [&](int64_t a, int64_t b) { return cost(a) > cost(b); });
  constexpr int kXcdCus = 32;
  size_t large = 0;   // events of more than a quarter of a bin's share: the first 32 at most
  if (deal) {
    int64_t total = 0;
    for (int64_t k : order) total += cost(k);
    while (large < order.size() && cost(order[large]) > total / (4 * kAttnBins)) ++large;
  }
  std::vector<int> bin_of(order.size());   // -1: dealt
  std::vector<int> tile_bin;               // bins of the dealt events' tiles
  int64_t load[kAttnBins] = {0};
  int64_t cnt[kAttnBins] = {0};
  auto assign = [&](int64_t c, int64_t t) {
    int best = 0;
    for (int b = 1; b < kAttnBins; ++b)
      if (load[b] < load[best]) best = b;
    load[best] += c;
    cnt[best] += t;
    return best;
  };
  for (size_t i = 0; i < order.size(); ++i) {
    const int64_t k = order[i];
    if (i < large && tiles(k) * deal > 2 * kXcdCus) {
      bin_of[i] = -1;
      for (int64_t q = 0; q < tiles(k); ++q) tile_bin.push_back(assign(nk(k), 1));
    } else {
      bin_of[i] = assign(cost(k), tiles(k));
    }
  }
  int64_t pos = 0;
  auto put = [&](int64_t k, int64_t q) {
    items[pos++] = AttnItem{(int32_t)(q_off[ids[k]] + q * qt),
                            (int32_t)std::min<int64_t>(qt, nq(k) - q * qt), (int32_t)k0(k),
                            (int32_t)nk(k)};
  };
  bins->max_len = 0;
  for (int b = 0; b < kAttnBins; ++b) {
    bins->start[b] = (int32_t)pos;
    bins->len[b] = (int32_t)cnt[b];
    bins->max_len = std::max<int32_t>(bins->max_len, (int32_t)cnt[b]);
    size_t dealt = 0;
    for (size_t i = 0; i < large; ++i)
      for (int64_t q = 0; bin_of[i] < 0 && q < tiles(order[i]); ++q)
        if (tile_bin[dealt++] == b) put(order[i], q);
    for (size_t i = 0; i < order.size(); ++i) {
      if (bin_of[i] != b) continue;
      for (int64_t q = 0; q < tiles(order[i]); ++q) put(order[i], q);
    }
  }
  return pos;
}
}  // namespace

int64_t build_attention_work(const int64_t* q_off, const int64_t* kv_off, const int64_t* ids,
                             int64_t n, int qt, int deal, AttnItem* items, AttnBins* bins) {
  return build_work(
      q_off, ids, n, qt, deal, [&](int64_t k) { return q_off[ids[k] + 1] - q_off[ids[k]]; },
      [&](int64_t k) { return kv_off[ids[k]]; },
      [&](int64_t k) { return kv_off[ids[k] + 1] - kv_off[ids[k]]; }, items, bins);
}

int64_t build_attention_work_kv(const int64_t* q_off, const int64_t* kv_start,
                                const int64_t* kv_len, const int64_t* ids, int64_t n, int qt,
                                int deal, AttnItem* items, AttnBins* bins) {
  return build_work(
      q_off, ids, n, qt, deal, [&](int64_t k) { return q_off[ids[k] + 1] - q_off[ids[k]]; },
      [&](int64_t k) { return kv_start[ids[k]]; }, [&](int64_t k) { return kv_len[ids[k]]; },
      items, bins);
}

int attention_query_tile(bool bf16, int dh, int64_t rows) {
  if (dh != kH32) return QT;
  // FP32: 128 queries share each staged (and split) chunk; below 32 items of 64 queries an
  // XCD and head the work is too thin for that and 64 spread it wider (632 rows: 11.7 us a launch with 64, 15.6
  // with 128; 14,276 rows: 30.2 and 30.5; 58,499 rows: 99 and 90; three tiles a wave spill)
  return bf16 || rows > 16384 ? 128 : 64;
}

// The FP32 kernel of heads of 32 takes several times as long as the BF16 one for the same keys, so
// one event on one XCD (32 of the 256 CUs) is the launch's time where a few large events make up
// a call. Their tiles go to all XCDs, which then read the keys from the last-level cache each (one
// event of 4,000, 8 heads: 858 us a launch whole, 143 dealt; the general kernel before: 230). Events
// that do not fill an XCD stay whole and read their keys from one L2 (60 events of 20-200, 8 heads:
// 19.5 us a launch whole, 20.2 with the larger ones dealt).
int attention_deal(bool bf16, int dh, int n_heads) { return !bf16 && dh == kH32 ? n_heads : 0; }

int attention_query_tiles(bool bf16, int dh, int* tiles) {
  if (bf16 && dh == kH32) {
    tiles[0] = 64;    // one 16-query tile per wave
    tiles[1] = 128;   // two
    tiles[2] = 192;   // three: events of up to 192 slots in one item (one workgroup per head)
    return 3;
  }
  tiles[0] = QT;
  return 1;
}

template <typename T>
hipError_t launch_attention(hipStream_t st, bool cross, int dh, int n_heads, int qt,
                            int64_t n_items, const AttnBins& bins, const AttnItem* work, const T* Q, int ldq,
                            int64_t hsq, const T* K, const T* V, int ldkv, int64_t hskv, T* O,
                            int ldo, int64_t hso, L2Touch touch) {
  if (n_items <= 0) return hipSuccess;
  if (n_items > 0x7fffffff) return hipErrorInvalidValue;
  const float sl2e = 1.4426950408889634f / sqrtf((float)dh);
  if (dh == kH32) {
    // 16-byte row chunks: row pitches and head offsets are multiples of 8 elements
    if (ldq % 8 || ldkv % 8 || ldo % 4 || hsq % 8 || hskv % 8 || hso % 4 || hsq < dh ||
        hskv < dh || hso < dh || (qt != 64 && qt != 128 && (qt != 192 || sizeof(T) == 4)))
      return hipErrorInvalidValue;
    // The grid holds every bin's items times the heads. A launch has at most 2^32 - 1 work items,
    // which millions of small events exceed (the runtime drops the excess without an error): then
    // a part of every bin at a time.
    const int64_t step = 0xffffffff / 256 / ((int64_t)kAttnBins * n_heads);
    auto parts = [&](auto&& launch) {
      for (int64_t i = 0; i < bins.max_len; i += step) {
        AttnBins part = bins;
        for (int b = 0; b < kAttnBins; ++b) {
          part.len[b] = (int32_t)std::min(step, std::max<int64_t>(bins.len[b] - i, 0));
          part.start[b] = (int32_t)(bins.start[b] + (part.len[b] ? i : 0));
        }
        part.max_len = (int32_t)std::min<int64_t>(step, bins.max_len - i);
        launch(part, (unsigned)(kAttnBins * part.max_len * n_heads));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
      }
      return hipSuccess;
    };
    if constexpr (std::is_same<T, bf16>::value) {
      // workgroups that read weights follow the attention part, a multiple of the XCD count (few
      // rows, so one launch)
      const int64_t warm = touch.p ? kAttnBins * ((touch.bytes + (int64_t)kTouchPart - 1) / kTouchPart) : 0;
      if (warm && (bins.max_len > step || kAttnBins * bins.max_len * n_heads + warm > 0xffffffff / 256))
        return hipErrorInvalidValue;
      auto go = [&](auto* k) {
        return parts([&](const AttnBins& part, unsigned blocks) {
          touch.first = blocks;
          hipLaunchKernelGGL(k, dim3(blocks + (unsigned)warm), dim3(256), 0, st, Q, ldq, hsq, K, V, ldkv,
                             hskv, O, ldo, hso, work, part, n_heads, sl2e, touch);
        });
      };
      if (cross) return go(qt == 64 ? k_attn32_cross<1> : qt == 128 ? k_attn32_cross<2> : k_attn32_cross<3>);
      return go(qt == 64 ? k_attn32_self<1> : qt == 128 ? k_attn32_self<2> : k_attn32_self<3>);
    } else {
      auto go = [&](auto* k) {
        return parts([&](const AttnBins& part, unsigned blocks) {
          hipLaunchKernelGGL(k, dim3(blocks), dim3(256), 0, st, Q, ldq, hsq, K, V, ldkv, hskv, O, ldo,
                             hso, work, part, n_heads, sl2e);
        });
      };
      if (cross) return go(qt == 64 ? k_attn_cross<1> : k_attn_cross<2>);
      return go(qt == 64 ? k_attn_self<1> : k_attn_self<2>);
    }
  }
  // the general kernel takes row-major operands only, in work items of QT queries
  if (hsq != dh || hskv != dh || hso != dh || qt != QT) return hipErrorInvalidValue;
  const dim3 grid((unsigned)n_items, n_heads);
  switch (dh) {
    case 16: return go_attn<T, 16>(cross, grid, st, Q, ldq, K, V, ldkv, O, ldo, work, sl2e);
    case 64: return go_attn<T, 64>(cross, grid, st, Q, ldq, K, V, ldkv, O, ldo, work, sl2e);
    default: return hipErrorInvalidValue;
  }
}

template hipError_t launch_attention<float>(hipStream_t, bool, int, int, int, int64_t,
                                            const AttnBins&, const AttnItem*, const float*, int,
                                            int64_t, const float*, const float*, int, int64_t,
                                            float*, int, int64_t, L2Touch);
template hipError_t launch_attention<bf16>(hipStream_t, bool, int, int, int, int64_t,
                                           const AttnBins&, const AttnItem*, const bf16*, int,
                                           int64_t, const bf16*, const bf16*, int, int64_t,
                                           bf16*, int, int64_t, L2Touch);

}  // namespace fmd
