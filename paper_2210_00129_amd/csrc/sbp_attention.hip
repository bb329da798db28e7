// Backward of scaled dot-product attention on the kept tokens (paper: main text section Design Strategies,
// "How to apply SBP on MHSA?", variant "Drop QKV"; supplement section Gradient Calculation of Attention
// Layers, eq:grad_qkv with the gradient dropout of eq:sbp_sep_on_query / eq:sbp_sep_on_key applied to dropped
// queries AND dropped keys).  Per sample and head, over the kept tokens i, j only:
//   S_ij  = exp(scale q_i.k_j - lse_i)          lse_i: log-sum-exp of the forward over ALL keys
//   dV_j  = sum_i S_ij dA_i
//   dM_ij = S_ij (dA_i.v_j - dA_i.A_i)          the softmax row term sum_l S_il dS_il equals dA_i.A_i (A = S V)
//   dQ_i  = scale sum_j dM_ij k_j,   dK_j = scale sum_i dM_ij q_i
// Kernels: for bf16 an MFMA kernel with one workgroup per sample and head (all kept tokens of the head in LDS) and a tiled one
// for any number of tokens; for fp32 tensors a tiled one on the fp32 matrix cores; a plain kernel for d = 16.
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <type_traits>

#include "sbp_internal.h"
#include "sbp_mfma_gemm.h"

namespace sbp {

static constexpr float kLog2e = 1.4426950408889634f;

// ------------------------------------------------------------------------------------------------
// plain kernel: an "owner" token per group of d/16 lanes; PHASE 0 owns a key (dK, dV, loop over the
// queries), PHASE 1 owns a query (dQ, loop over the keys).  Sums run in token order: deterministic.
// ------------------------------------------------------------------------------------------------
template <typename T> struct AtIO;
template <> struct AtIO<uint16_t> {
  static __device__ __forceinline__ void load16(const uint16_t* p, float (&v)[16]) {
    const uint4 a = reinterpret_cast<const uint4*>(p)[0], b = reinterpret_cast<const uint4*>(p)[1];
    const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
    for (int i = 0; i < 8; ++i) { v[2 * i] = bf16_lo(w[i]); v[2 * i + 1] = bf16_hi(w[i]); }
  }
  static __device__ __forceinline__ void store16(uint16_t* p, const float (&v)[16]) {
    uint32_t w[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = bf16_pack(v[2 * i], v[2 * i + 1]);
    reinterpret_cast<uint4*>(p)[0] = make_uint4(w[0], w[1], w[2], w[3]);
    reinterpret_cast<uint4*>(p)[1] = make_uint4(w[4], w[5], w[6], w[7]);
  }
};
template <> struct AtIO<float> {
  static __device__ __forceinline__ void load16(const float* p, float (&v)[16]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float4 a = reinterpret_cast<const float4*>(p)[i];
      v[4 * i] = a.x; v[4 * i + 1] = a.y; v[4 * i + 2] = a.z; v[4 * i + 3] = a.w;
    }
  }
  static __device__ __forceinline__ void store16(float* p, const float (&v)[16]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) reinterpret_cast<float4*>(p)[i] = make_float4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
  }
};

__device__ __forceinline__ float dot16(const float (&a)[16], const float (&b)[16]) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) s = fmaf(a[i], b[i], s);
  return s;
}
__device__ __forceinline__ float group_sum(float v, int lanes) {   // over `lanes` (1, 2, 4 or 8) adjacent lanes
  for (int m = 1; m < lanes; m <<= 1) v += __shfl_xor(v, m);
  return v;
}

template <typename T, int PHASE>
__global__ void __launch_bounds__(256) attn_bwd_plain_kernel(const T* __restrict__ qkv, const T* __restrict__ A,
                                                              const T* __restrict__ dA, const float* __restrict__ lse,
                                                              int n_k, int h, int d, float scale, T* __restrict__ dqkv) {
  const int cper = d / 16, owners = 256 / cper;
  const int o = blockIdx.x * owners + (int)threadIdx.x / cper, c = (int)threadIdx.x % cper;
  const int head = blockIdx.y, b = blockIdx.z;
  const int tok = min(o, n_k - 1);
  const long long row0 = (long long)b * n_k, ldq = 3LL * h * d, lda = (long long)h * d;
  const int col = head * d + 16 * c;
  const T* q_base = qkv + col;
  const T* k_base = qkv + (long long)h * d + col;
  const T* v_base = qkv + 2LL * h * d + col;
  float own1[16], own2[16], acc1[16], acc2[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc1[i] = acc2[i] = 0.f;
  if (PHASE == 0) {
    AtIO<T>::load16(k_base + (row0 + tok) * ldq, own1);
    AtIO<T>::load16(v_base + (row0 + tok) * ldq, own2);
    for (int t = 0; t < n_k; ++t) {
      float q[16], g[16], a[16];
      AtIO<T>::load16(q_base + (row0 + t) * ldq, q);
      AtIO<T>::load16(dA + (row0 + t) * lda + col, g);
      AtIO<T>::load16(A + (row0 + t) * lda + col, a);
      const float s = group_sum(dot16(q, own1), cper);
      const float dp = group_sum(dot16(g, own2), cper);
      const float delta = group_sum(dot16(g, a), cper);
      const float p = expf(scale * s - lse[(row0 + t) * h + head]);
      const float ds = p * (dp - delta) * scale;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        acc2[i] = fmaf(p, g[i], acc2[i]);       // dV_j += S_ij dA_i
        acc1[i] = fmaf(ds, q[i], acc1[i]);      // dK_j += scale dM_ij q_i
      }
    }
    if (o < n_k) {
      AtIO<T>::store16(dqkv + (row0 + o) * ldq + (long long)h * d + col, acc1);
      AtIO<T>::store16(dqkv + (row0 + o) * ldq + 2LL * h * d + col, acc2);
    }
  } else {
    float a[16];
    AtIO<T>::load16(q_base + (row0 + tok) * ldq, own1);
    AtIO<T>::load16(dA + (row0 + tok) * lda + col, own2);
    AtIO<T>::load16(A + (row0 + tok) * lda + col, a);
    const float delta = group_sum(dot16(own2, a), cper);
    const float l = lse[(row0 + tok) * h + head];
    for (int t = 0; t < n_k; ++t) {
      float k[16], v[16];
      AtIO<T>::load16(k_base + (row0 + t) * ldq, k);
      AtIO<T>::load16(v_base + (row0 + t) * ldq, v);
      const float s = group_sum(dot16(own1, k), cper);
      const float dp = group_sum(dot16(own2, v), cper);
      const float p = expf(scale * s - l);
      const float ds = p * (dp - delta) * scale;
#pragma unroll
      for (int i = 0; i < 16; ++i) acc1[i] = fmaf(ds, k[i], acc1[i]);   // dQ_i += scale dM_ij k_j
    }
    if (o < n_k) AtIO<T>::store16(dqkv + (row0 + o) * ldq + col, acc1);
  }
}

// ------------------------------------------------------------------------------------------------
// MFMA kernel (bf16).  One workgroup of 4 wavefronts per (sample, head).  LDS: the kept rows of q, k, v
// and dA of the head as [NPAD][D] tiles (rows padded with zeros to a multiple of 32, pitch 2 D + 16
// bytes: 16-byte reads of 16 consecutive rows and the transposing reads hit distinct banks), and the
// per-token tables lse * log2(e) and delta = dA.A.
//
// v_mfma_f32_32x32x16_bf16 register layouts (lane l, u = l >> 5):  A[row l & 31][k 8u .. 8u+7],
// B[k 8u .. 8u+7][col l & 31],  C register v = C[row 8 (v >> 2) + 4u + (v & 3)][col l & 31].
// Phase 1, wavefront = block of 32 keys j, loop over blocks of 32 queries i:
//   S = Q_i K_j^T and dP = dA_i V_j^T   (operands: 16-byte row reads, contraction over the head dim)
//   P = exp2(S c - lse_i),  dS = P (dP - delta_i)          in the C layout: rows i, column j = lane
//   dV_j^T += dA_i^T P,  dK_j^T += Q_i^T dS                 contraction over i: C registers 8 ks .. 8 ks + 7
//     hold rows 16 ks + 4u + (0..3) and 16 ks + 8 + 4u + (0..3) of the lane's column, which is a valid B
//     operand if the A operand lists the same rows: two ds_read_b64_tr_b16 of those 4 + 4 token rows.
// Phase 2, wavefront = block of 32 queries i, loop over blocks of keys j: the transposes S^T = K_j Q_i^T,
//   dP^T = V_j dA_i^T (lse_i and delta_i are then per-lane scalars), dQ_i^T += K_j^T dS^T.
// Recomputing S and dP in phase 2 costs 2 of 7 products and saves every cross-wavefront reduction:
// results are deterministic.  Padded rows are zero, so padded queries add nothing (dA = 0, delta = 0) and
// padded keys add nothing to dQ (k = 0); their own outputs are not stored.
// ------------------------------------------------------------------------------------------------
template <int D>
struct AttnLds {
  static constexpr int PITCH = 2 * D + 16;
  static __host__ __device__ size_t bytes(int npad) { return (size_t)4 * npad * PITCH + (size_t)2 * npad * sizeof(float); }
};

__device__ __forceinline__ bf16x8_t pack8(const f32x16_t& c, int ks) {
  uint32_t w[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) w[e] = bf16_pack(c[8 * ks + 2 * e], c[8 * ks + 2 * e + 1]);
  return __builtin_bit_cast(bf16x8_t, make_uint4(w[0], w[1], w[2], w[3]));
}

// Two LDS layouts of a tile of token rows, each with the lane's two kinds of operand reads:
//   row(tile, row0, ks): 16 bytes of row row0 + (lane & 31), head dimensions 16 ks + 8 u .. + 7
//   tr(tile, row0, x):   A operand [head dimensions 32 x .. + 31][16 tokens]: token rows row0 + 4u + (0..3) and
//                        row0 + 8 + 4u + (0..3) (two transposing reads; row0 is a multiple of 16)
// AttnPadded: rows of 2 D + 16 bytes, written from registers.
template <int D>
struct AttnPadded {
  static constexpr int PITCH = AttnLds<D>::PITCH;
  int foff, toff;
  __device__ __forceinline__ explicit AttnPadded(int lane) {
    const int g = lane >> 4, i = lane & 15;
    foff = (lane & 31) * PITCH + 16 * (lane >> 5);
    toff = (4 * (g >> 1) + (i >> 2)) * PITCH + (16 * (g & 1) + 4 * (i & 3)) * 2;
  }
  __device__ __forceinline__ bf16x8_t row(const char* tile, int row0, int ks) const {
    return *reinterpret_cast<const bf16x8_t*>(tile + row0 * PITCH + foff + ks * 32);
  }
  __device__ __forceinline__ bf16x8_t tr(const char* tile, int row0, int x) const {
    const char* p = tile + row0 * PITCH + toff + 64 * x;
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((SBP_LDS s16x4_t*)(p));
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((SBP_LDS s16x4_t*)(p + 8 * PITCH));
    return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
};
// AttnSwizzled: rows of 2 D bytes, 16-byte chunk c of row r at place c ^ swz(r), written by global -> LDS copies whose lanes
// choose the chunk they fetch (the copy fixes the LDS place by lane; a copy fills 1 KB, 512 / D rows).  By their addresses both
// kinds of reads meet all 64 banks once: a transposing read's half wavefront takes 64 bytes of each of 4 neighbouring rows, so these
// rows differ in the bits of the place above the chunks it takes (bit 2; D = 128: bits 2 and 3), and the 16-byte reads of 16
// neighbouring rows fall on different places because the copies within 16 rows lie 16 bytes further apart than their 1 KB (not for
// D = 32, whose 16 rows are one copy: rows r and r + 8 share banks, two turns).  That holds for 16 consecutive lanes to a turn; the
// counter still has conflicts in 31 % of the LDS cycles at D = 64, 44 before.  (With c ^ (r & 7) and no
// gaps rows r and r + 2 exchanged places within the same 64 bytes: every transposing read took two turns, D = 128 four.)
template <int D>
struct AttnSwizzled {
  static constexpr int RB = 2 * D, CH = D / 8, KS = D / 16, DB = D / 32;
  static constexpr int RPC = 512 / D, COPY = D == 32 ? 1024 : 1040, G16 = (16 / RPC - 1) * COPY + 1024;   // rows of a copy, pitch of the copies, bytes of 16 rows
  static __device__ __forceinline__ int swz(int r) {
    return D == 32 ? (r >> 1) & 3 : D == 64 ? (r & 2) << 1 | (r & 4) >> 1 : (r & 3) << 2;
  }
  static __device__ __forceinline__ int place(int r) { return (r >> 4) * G16 + ((r & 15) / RPC) * COPY + (r % RPC) * RB; }
  int foff[KS], toff[DB];
  __device__ __forceinline__ explicit AttnSwizzled(int lane) {
    const int g = lane >> 4, i = lane & 15, r = lane & 31, rt = 4 * (g >> 1) + (i >> 2);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) foff[ks] = place(r) + (((2 * ks + (lane >> 5)) ^ swz(r)) << 4);
#pragma unroll
    for (int x = 0; x < DB; ++x) toff[x] = place(rt) + (((4 * x + 2 * (g & 1) + ((i & 3) >> 1)) ^ swz(rt)) << 4) + 8 * (i & 1);
  }
  // row0: a multiple of 32
  __device__ __forceinline__ bf16x8_t row(const char* tile, int row0, int ks) const {
    return *reinterpret_cast<const bf16x8_t*>(tile + (row0 >> 4) * G16 + foff[ks]);
  }
  // row0: a multiple of 16; rows 8 further on lie 8 / RPC copies further on, with the same swz
  __device__ __forceinline__ bf16x8_t tr(const char* tile, int row0, int x) const {
    const char* p = tile + (row0 >> 4) * G16 + toff[x];
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((SBP_LDS s16x4_t*)(p));
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((SBP_LDS s16x4_t*)(p + (D == 32 ? 8 * RB : 8 / RPC * COPY)));
    return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
};

// The LDS image of one (sample, head): four tiles and two tables.
template <int D>
struct AttnTiles {
  static constexpr int PITCH = AttnLds<D>::PITCH;
  char *tq, *tk, *tv, *tg;       // q, k, v, dA
  float *lse_s, *delta_s;        // lse * log2(e), -dA.A
  __device__ __forceinline__ void place(char* base, int npad) {
    tq = base;
    tk = tq + npad * PITCH;
    tv = tk + npad * PITCH;
    tg = tv + npad * PITCH;
    lse_s = reinterpret_cast<float*>(tg + npad * PITCH);
    delta_s = lse_s + npad;
  }
};

// Where one (sample, head) lives in global memory.
struct AttnItem {
  const uint16_t *q, *a, *g;     // row 0 of the head's columns in qkv (q third), A and dA
  const float* lse;              // lse[row 0][head]
  uint16_t* o;                   // row 0 of the head's columns in dqkv (dQ third)
};
__device__ __forceinline__ AttnItem attn_item(const uint16_t* qkv, const uint16_t* A, const uint16_t* dA, const float* lse,
                                              uint16_t* dqkv, int b, int head, int n_k, int h, int D) {
  const long long row0 = (long long)b * n_k;
  AttnItem it;
  it.q = qkv + row0 * (3LL * h * D) + head * D;
  it.a = A + row0 * ((long long)h * D) + head * D;
  it.g = dA + row0 * ((long long)h * D) + head * D;
  it.lse = lse + row0 * h + head;
  it.o = dqkv + row0 * (3LL * h * D) + head * D;
  return it;
}

// R rounds of 16-byte pieces per thread (NT threads): piece p = token p / CH, chunk p % CH of q, k, v, dA and A.
template <int D, int R>
struct AttnPieces {
  uint4 q[R], k[R], v[R], g[R], a[R];
  template <int NT>
  __device__ __forceinline__ void load(const AttnItem& it, int p0, int n_k, int h) {
    constexpr int CH = D / 8;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int p = p0 + NT * r, tok = p / CH, ch = p % CH;
      q[r] = k[r] = v[r] = g[r] = a[r] = make_uint4(0, 0, 0, 0);
      if (tok < n_k) {                                   // also false for pieces past the padded tile
        const uint16_t* src = it.q + (long long)tok * (3LL * h * D) + 8 * ch;
        q[r] = *reinterpret_cast<const uint4*>(src);
        k[r] = *reinterpret_cast<const uint4*>(src + (long long)h * D);
        v[r] = *reinterpret_cast<const uint4*>(src + 2LL * h * D);
        g[r] = *reinterpret_cast<const uint4*>(it.g + (long long)tok * ((long long)h * D) + 8 * ch);
        a[r] = *reinterpret_cast<const uint4*>(it.a + (long long)tok * ((long long)h * D) + 8 * ch);
      }
    }
  }
  template <int NT>
  __device__ __forceinline__ void store(const AttnTiles<D>& T, int p0, int npieces) const {
    constexpr int CH = D / 8, PITCH = AttnLds<D>::PITCH;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int p = p0 + NT * r, tok = p / CH, ch = p % CH;
      if (p < npieces) {                                 // uniform per wavefront: npieces is a multiple of 64
        const int off = tok * PITCH + ch * 16;
        *reinterpret_cast<uint4*>(T.tq + off) = q[r];
        *reinterpret_cast<uint4*>(T.tk + off) = k[r];
        *reinterpret_cast<uint4*>(T.tv + off) = v[r];
        *reinterpret_cast<uint4*>(T.tg + off) = g[r];
        const uint32_t gw[4] = {g[r].x, g[r].y, g[r].z, g[r].w}, aw[4] = {a[r].x, a[r].y, a[r].z, a[r].w};
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) s += bf16_lo(gw[e]) * bf16_lo(aw[e]) + bf16_hi(gw[e]) * bf16_hi(aw[e]);
        for (int m = 1; m < CH; m <<= 1) s += __shfl_xor(s, m);
        if (ch == 0) T.delta_s[tok] = -s;
      }
    }
  }
};

// dK and dV of 32 keys (one wavefront): the keys' fragments live in registers, the queries come block by block from
// LDS tiles (tq, tg: rows of q and dA; lse_s, delta_s: their tables), any number of tiles one after the other.
template <int D>
struct AttnKeyAcc {
  static constexpr int PITCH = AttnLds<D>::PITCH, KS = D / 16, DB = D / 32;
  f32x16_t dv[DB], dk[DB];
  bf16x8_t kf[KS], vf[KS];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int x = 0; x < DB; ++x)
#pragma unroll
      for (int e = 0; e < 16; ++e) dv[x][e] = dk[x][e] = 0.f;
  }
  // fragments of the keys from LDS tiles (rows row0 .. row0 + 31)
  __device__ __forceinline__ void keys_from_lds(const char* tk, const char* tv, int row0, int lane) {
    const int foff = (row0 + (lane & 31)) * PITCH + 16 * (lane >> 5);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      kf[ks] = *reinterpret_cast<const bf16x8_t*>(tk + foff + ks * 32);
      vf[ks] = *reinterpret_cast<const bf16x8_t*>(tv + foff + ks * 32);
    }
  }
  // ... or straight from memory: k and v of the lane's token (row pointers of the head's columns)
  __device__ __forceinline__ void from_memory(const uint16_t* krow, const uint16_t* vrow, int lane) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      kf[ks] = *reinterpret_cast<const bf16x8_t*>(krow + 16 * ks + 8 * (lane >> 5));
      vf[ks] = *reinterpret_cast<const bf16x8_t*>(vrow + 16 * ks + 8 * (lane >> 5));
    }
  }
  // dP starts from -delta (read straight into the accumulators), so that dS = P dP needs no subtraction
  template <class L>
  __device__ __forceinline__ void run(const L& lay, const char* tq, const char* tg, const float* lse_s, const float* delta_s, int nblk,
                                      float scale, int lane) {
    const int u = lane >> 5;
    const float c2 = scale * kLog2e;
    for (int ib = 0; ib < nblk; ++ib) {
      f32x16_t s, dp;
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const f32x4_t d4 = *reinterpret_cast<const f32x4_t*>(delta_s + ib * 32 + 8 * q4 + 4 * u);
#pragma unroll
        for (int e = 0; e < 4; ++e) { dp[4 * q4 + e] = d4[e]; s[4 * q4 + e] = 0.f; }
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lay.row(tq, ib * 32, ks), kf[ks], s, 0, 0, 0);      // rows i, columns j
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lay.row(tg, ib * 32, ks), vf[ks], dp, 0, 0, 0);
      }
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const f32x4_t l4 = *reinterpret_cast<const f32x4_t*>(lse_s + ib * 32 + 8 * q4 + 4 * u);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float p = __builtin_amdgcn_exp2f(s[4 * q4 + e] * c2 - l4[e]);
          s[4 * q4 + e] = p;
          dp[4 * q4 + e] *= p;
        }
      }
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const bf16x8_t pf = pack8(s, ks), dsf = pack8(dp, ks);
#pragma unroll
        for (int x = 0; x < DB; ++x) {
          dv[x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lay.tr(tg, ib * 32 + 16 * ks, x), pf, dv[x], 0, 0, 0);   // rows head dim, columns j
          dk[x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lay.tr(tq, ib * 32 + 16 * ks, x), dsf, dk[x], 0, 0, 0);
        }
      }
    }
  }
  // key j = first key of the block + (lane & 31); out: row 0 of the head's columns in dqkv
  __device__ __forceinline__ void store(uint16_t* __restrict__ out, int j, int n_k, int h, float scale, int lane) const {
    const int u = lane >> 5;
    if (j < n_k) {
      uint16_t* o = out + (long long)j * (3LL * h * D);
#pragma unroll
      for (int x = 0; x < DB; ++x)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int dcol = 32 * x + 8 * q4 + 4 * u;
          uint2 w;
          w.x = bf16_pack(dk[x][4 * q4] * scale, dk[x][4 * q4 + 1] * scale);
          w.y = bf16_pack(dk[x][4 * q4 + 2] * scale, dk[x][4 * q4 + 3] * scale);
          *reinterpret_cast<uint2*>(o + (long long)h * D + dcol) = w;
          w.x = bf16_pack(dv[x][4 * q4], dv[x][4 * q4 + 1]);
          w.y = bf16_pack(dv[x][4 * q4 + 2], dv[x][4 * q4 + 3]);
          *reinterpret_cast<uint2*>(o + 2LL * h * D + dcol) = w;
        }
    }
  }
};

// dQ of 32 queries (one wavefront): the queries' fragments, lse and delta live in registers, the keys come block by
// block from LDS tiles (tk, tv).
template <int D>
struct AttnQueryAcc {
  static constexpr int PITCH = AttnLds<D>::PITCH, KS = D / 16, DB = D / 32;
  f32x16_t dq[DB];
  bf16x8_t qf[KS], gf[KS];
  float l;                       // lse * log2(e) of query (lane & 31)
  f32x16_t nd;                   // -delta of that query in every register: dP starts from it
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int x = 0; x < DB; ++x)
#pragma unroll
      for (int e = 0; e < 16; ++e) dq[x][e] = 0.f;
  }
  __device__ __forceinline__ void queries_from_lds(const char* tq, const char* tg, const float* lse_s, const float* delta_s,
                                                   int row0, int lane) {
    const int foff = (row0 + (lane & 31)) * PITCH + 16 * (lane >> 5);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      qf[ks] = *reinterpret_cast<const bf16x8_t*>(tq + foff + ks * 32);
      gf[ks] = *reinterpret_cast<const bf16x8_t*>(tg + foff + ks * 32);
    }
    l = lse_s[row0 + (lane & 31)];
    start(delta_s[row0 + (lane & 31)]);
  }
  __device__ __forceinline__ void start(float ndl) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      nd[e] = ndl;
      asm("" : "+v"(nd[e]));                   // (16 registers for good: as one value it would be copied 16 times per block)
    }
  }
  // straight from memory: q, dA, A rows of the lane's token (head's columns) and its lse
  __device__ __forceinline__ void from_memory(const uint16_t* qrow, const uint16_t* grow, const uint16_t* arow, const float* lse_tok, int lane) {
    float part = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      qf[ks] = *reinterpret_cast<const bf16x8_t*>(qrow + 16 * ks + 8 * (lane >> 5));
      const uint4 b = *reinterpret_cast<const uint4*>(grow + 16 * ks + 8 * (lane >> 5)), c = *reinterpret_cast<const uint4*>(arow + 16 * ks + 8 * (lane >> 5));
      gf[ks] = __builtin_bit_cast(bf16x8_t, b);
      const uint32_t gw[4] = {b.x, b.y, b.z, b.w}, aw[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) part += bf16_lo(gw[e]) * bf16_lo(aw[e]) + bf16_hi(gw[e]) * bf16_hi(aw[e]);
    }
    start(-(part + __shfl_xor(part, 32)));     // the two halves of every 16 columns lie 32 lanes apart
    l = *lse_tok * kLog2e;
  }
  // keys: valid rows of the tile (rows past them count for nothing: their probabilities are zeroed)
  template <class L>
  __device__ __forceinline__ void run(const L& lay, const char* tk, const char* tv, int keys, float scale, int lane) {
    int j0 = 0;
    for (; j0 + 32 <= keys; j0 += 32) block<false>(lay, tk, tv, j0, keys, scale, lane);
    if (j0 < keys) block<true>(lay, tk, tv, j0, keys, scale, lane);
  }
  template <bool TAIL, class L>
  __device__ __forceinline__ void block(const L& lay, const char* tk, const char* tv, int j0, int keys, float scale, int lane) {
    const float c2 = scale * kLog2e;
    f32x16_t s, dp;
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lay.row(tk, j0, ks), qf[ks], s, 0, 0, 0);      // rows j, columns i
      dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lay.row(tv, j0, ks), gf[ks], ks ? dp : nd, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) dp[e] *= __builtin_amdgcn_exp2f(s[e] * c2 - l);
    if constexpr (TAIL) {
#pragma unroll
      for (int e = 0; e < 16; ++e) dp[e] = j0 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3) < keys ? dp[e] : 0.f;
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const bf16x8_t dsf = pack8(dp, ks);
#pragma unroll
      for (int x = 0; x < DB; ++x)
        dq[x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lay.tr(tk, j0 + 16 * ks, x), dsf, dq[x], 0, 0, 0);   // rows head dim, columns i
    }
  }
  __device__ __forceinline__ void store(uint16_t* __restrict__ out, int i, int n_k, int h, float scale, int lane) const {
    const int u = lane >> 5;
    if (i < n_k) {
      uint16_t* o = out + (long long)i * (3LL * h * D);
#pragma unroll
      for (int x = 0; x < DB; ++x)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          uint2 w;
          w.x = bf16_pack(dq[x][4 * q4] * scale, dq[x][4 * q4 + 1] * scale);
          w.y = bf16_pack(dq[x][4 * q4 + 2] * scale, dq[x][4 * q4 + 3] * scale);
          *reinterpret_cast<uint2*>(o + 32 * x + 8 * q4 + 4 * u) = w;
        }
    }
  }
};

template <int D>
__device__ __forceinline__ void attn_key_block(const AttnTiles<D>& T, int jb, int nblk, int n_k, int h, float scale,
                                               uint16_t* __restrict__ out, int lane) {
  AttnKeyAcc<D> acc;
  acc.zero();
  acc.keys_from_lds(T.tk, T.tv, jb * 32, lane);
  acc.run(AttnPadded<D>(lane), T.tq, T.tg, T.lse_s, T.delta_s, nblk, scale, lane);
  acc.store(out, jb * 32 + (lane & 31), n_k, h, scale, lane);
}

template <int D>
__device__ __forceinline__ void attn_query_block(const AttnTiles<D>& T, int ib, int n_k, int h, float scale,
                                                 uint16_t* __restrict__ out, int lane) {
  AttnQueryAcc<D> acc;
  acc.zero();
  acc.queries_from_lds(T.tq, T.tg, T.lse_s, T.delta_s, ib * 32, lane);
  acc.run(AttnPadded<D>(lane), T.tk, T.tv, n_k, scale, lane);
  acc.store(out, ib * 32 + (lane & 31), n_k, h, scale, lane);
}

// One (sample, head) per workgroup of 4 wavefronts: load, then the key blocks, then the query blocks.  Any
// number of kept tokens whose tiles fit LDS.
template <int D>
__global__ void __launch_bounds__(256, D == 128 ? 1 : 2) attn_bwd_mfma_kernel(const uint16_t* __restrict__ qkv, const uint16_t* __restrict__ A,
                                                             const uint16_t* __restrict__ dA, const float* __restrict__ lse,
                                                             int n_k, int h, float scale, uint16_t* __restrict__ dqkv) {
  constexpr int CH = D / 8;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int npad = (n_k + 31) & ~31, nblk = npad >> 5;
  AttnTiles<D> T;
  T.place(smem, npad);
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const AttnItem it = attn_item(qkv, A, dA, lse, dqkv, blockIdx.y, blockIdx.x, n_k, h, D);
  const int npieces = npad * CH;
  for (int p0 = t; p0 < npieces; p0 += 4 * 256) {      // four rounds of loads in flight per thread
    AttnPieces<D, 4> pc;
    pc.template load<256>(it, p0, n_k, h);
    pc.template store<256>(T, p0, npieces);
  }
  for (int i = t; i < npad; i += 256) T.lse_s[i] = i < n_k ? it.lse[(long long)i * h] * kLog2e : 0.f;
  __syncthreads();
  for (int jb = wave; jb < nblk; jb += 4) attn_key_block<D>(T, jb, nblk, n_k, h, scale, it.o, lane);
  for (int ib = wave; ib < nblk; ib += 4) attn_query_block<D>(T, ib, n_k, h, scale, it.o, lane);
}

// ------------------------------------------------------------------------------------------------
// Tiled MFMA kernel: any number of kept tokens.  A workgroup of 4 wavefronts owns a chunk of 128 tokens of one (sample,
// head) in one of two roles: as keys (dK, dV; every wavefront holds the k and v fragments of its 32 keys in registers, the
// queries - rows of q and dA, lse, -delta - stream through LDS in tiles of 64) or as queries (dQ; q, dA fragments, lse,
// -delta in registers, rows of k and v stream).  Every output element is written by exactly one wavefront, sums run in token
// order: deterministic, no atomics.
// A ring of three tiles is filled by global -> LDS copies that are issued two tiles ahead, but every stage begins by waiting for
// all copies under way, so that a tile has the products of one other tile to arrive in.  The key role makes -delta and lse tables
// of 512 queries at a time from memory, so that its loop holds nothing but fragments and accumulators: 168 registers, three
// workgroups per CU.  (A spilled register in the loop waits, loads being counted in order, for the copies under way: with
// 17 of them the launch took 148 us.)  dP starts from -delta in the accumulators.  Rows past n_k are copies of the last row:
// as queries their lse is so large that their probabilities are 0, as keys their probabilities are zeroed (peeled block).
// The outputs leave through LDS as whole rows.  The workgroups of a (sample, head) run on one XCD, whose L2 they share
// (8 x 12 heads of 1024 tokens, counters: 289 MB read and 41 written across the L2 boundary by the kernel before, spread over all
// eight; now 60 and 38); an XCD runs its key units first, the longer kind (110 -> 102 us), at the price of a second read of small
// heads (27.6 instead of 26.6 us at 768 heads of 99 tokens).
// Bound, by counters: the matrix cores are busy 47 % of the cycles of a CU, the LDS 46 % (55 % with the layout before,
// AttnSwizzled; conflicts 31 and 44 % of that), and the softmax arithmetic between the products takes most of the rest; unit starts (first
// tiles and tables from memory) and the power limit (1.85 GHz) add to it.  8 x 12 heads of 64, 1024 kept tokens, a call:
// 134 -> 101 us with the ring, 99.6 with dP of the query role started from -delta and that layout; 8 x 12 heads of
// 32 62.9 -> 60.4 us; 8 x 8 heads of 128, whose transposing reads took four turns, 184 -> 163 us.  Both blocks of a tile unrolled
// (constant LDS addresses): 35 to 77 spills with three workgroups per CU, 114 us with two.  s_setprio around the products: 98.1 us, but
// 58.8 instead of 54.9 us at 64 x 12 heads of 197 tokens.
// Two more shapes were slower: 64 tokens per wavefront (half the LDS reads per MFMA, but 330 registers and one wavefront
// per SIMD: accumulator moves and spills, 225 us), and the same with dK and dV as separate roles (148 us).
// ------------------------------------------------------------------------------------------------
static constexpr int kAttnChunk = 128, kAttnTile = 64, kAttnRing = 3, kAttnTable = 512;

template <int D> struct AttnTiled {
  static constexpr int RB = 2 * D, IMG = kAttnTile / 16 * AttnSwizzled<D>::G16, STAGE = 2 * IMG;    // bytes per row, image, tile
  static constexpr size_t LDS = (size_t)kAttnRing * STAGE + 2 * kAttnTable * sizeof(float);
  static_assert(4 * 2 * 32 * (RB + 16) <= kAttnRing * STAGE, "the output images fit the ring");
};

__device__ __forceinline__ float attn_dot2(uint32_t a, uint32_t b, float c) {      // two exact products added in fp32
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), c, false);
}

// the streamed side: two images per tile, copied global -> LDS
template <int D>
struct AttnStream {
  static constexpr int CH = D / 8, RB = 2 * D, NI = D / 32;                  // 16-byte pieces and bytes per row, copies per wavefront and image
  const uint16_t *s1, *s2;             // q, dA or k, v
  uint32_t off1[NI], off2[NI];         // byte offsets of the lane's pieces in a tile
  int ld1, ld2, n_k;                   // row lengths
  __device__ __forceinline__ AttnStream(const uint16_t* s1_, const uint16_t* s2_, int ld1_, int ld2_, int n_k_, int lane, int wave)
      : s1(s1_), s2(s2_), ld1(ld1_), ld2(ld2_), n_k(n_k_) { offsets(kAttnTile, lane, wave); }
  __device__ __forceinline__ void offsets(int rows, int lane, int wave) {      // rows: valid rows of the tile; others copy the last one
#pragma unroll
    for (int n = 0; n < NI; ++n) {
      const int row = (wave * NI + n) * (1024 / RB) + lane / CH, c = (lane % CH) ^ AttnSwizzled<D>::swz(row);
      off1[n] = (uint32_t)min(row, rows - 1) * (uint32_t)ld1 * 2u + 16u * c;
      off2[n] = (uint32_t)min(row, rows - 1) * (uint32_t)ld2 * 2u + 16u * c;
    }
  }
  // copies of tile s (the tiles in order) into its ring place
  __device__ __forceinline__ void issue(int s, char* ring, int lane, int wave) {
    char* buf = ring + (s % kAttnRing) * AttnTiled<D>::STAGE + wave * AttnSwizzled<D>::G16;    // (a wavefront copies 16 rows)
    if ((s + 1) * kAttnTile > n_k) offsets(n_k - s * kAttnTile, lane, wave);
    const char* b1 = reinterpret_cast<const char*>(s1 + (long long)s * kAttnTile * ld1);
    const char* b2 = reinterpret_cast<const char*>(s2 + (long long)s * kAttnTile * ld2);
#pragma unroll
    for (int n = 0; n < NI; ++n) {
      async_copy16(b1 + off1[n], buf + n * AttnSwizzled<D>::COPY);
      async_copy16(b2 + off2[n], buf + AttnTiled<D>::IMG + n * AttnSwizzled<D>::COPY);
    }
  }
};

// Writes an accumulated [head dim][32 tokens] block to the tokens' rows (out: row 0 of the head's columns) through LDS
// (one 32-row image of the wavefront's own, pitch 2 D + 16 bytes): whole 2 D-byte rows instead of 8-byte pieces
template <int D>
__device__ __forceinline__ void attn_store_rows(char* image, const f32x16_t (&acc)[D / 32], float f, uint16_t* __restrict__ out, long long ld,
                                                int first, int n_k, int lane) {
  constexpr int PITCH = 2 * D + 16, LPR = D / 8;           // lanes per row
  char* row = image + (lane & 31) * PITCH + 8 * (lane >> 5);
#pragma unroll
  for (int x = 0; x < D / 32; ++x)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4)
      *reinterpret_cast<uint2*>(row + 64 * x + 16 * q4) = make_uint2(bf16_pack(acc[x][4 * q4] * f, acc[x][4 * q4 + 1] * f),
                                                                     bf16_pack(acc[x][4 * q4 + 2] * f, acc[x][4 * q4 + 3] * f));
#pragma unroll
  for (int r = 0; r < 32 * LPR / 64; ++r) {                // (a wavefront's LDS accesses complete in order)
    const int tok = r * (64 / LPR) + lane / LPR, c = lane % LPR;
    const uint4 v = *reinterpret_cast<const uint4*>(image + tok * PITCH + 16 * c);
    if (first + tok < n_k) *reinterpret_cast<uint4*>(out + (first + tok) * ld + 8 * c) = v;
  }
}

// lse * log2(e) and -delta = -dA.A of tokens t0 .. t0 + 511 (key role): four lanes per row, UNR rows in flight per lane
template <int D, int UNR>
__device__ __forceinline__ void attn_make_tables(const AttnItem& it, int t0, int n_k, int h, float* lse_s, float* ndl_s) {
  static_assert(kAttnTable % (64 * UNR) == 0, "whole rounds: every row that is written lies in the table");
  const int t = threadIdx.x, n = min(kAttnTable, n_k - t0);
  const long long lda = (long long)h * D;
  float lv[kAttnTable / 256];
#pragma unroll
  for (int i = 0; i < kAttnTable / 256; ++i) lv[i] = it.lse[(long long)min(t0 + t + 256 * i, n_k - 1) * h];
  for (int r0 = 0; r0 < n; r0 += 64 * UNR) {
    uint4 x[UNR][D / 32], y[UNR][D / 32];
#pragma unroll
    for (int v = 0; v < UNR; ++v) {
      const long long off = min(t0 + r0 + 64 * v + (t >> 2), n_k - 1) * lda + (t & 3) * (D / 4);
#pragma unroll
      for (int r = 0; r < D / 32; ++r) {
        x[v][r] = *reinterpret_cast<const uint4*>(it.g + off + 8 * r);
        y[v][r] = *reinterpret_cast<const uint4*>(it.a + off + 8 * r);
      }
    }
#pragma unroll
    for (int v = 0; v < UNR; ++v) {
      float d = 0.f;
#pragma unroll
      for (int r = 0; r < D / 32; ++r)
        d = attn_dot2(x[v][r].x, y[v][r].x, attn_dot2(x[v][r].y, y[v][r].y, attn_dot2(x[v][r].z, y[v][r].z, attn_dot2(x[v][r].w, y[v][r].w, d))));
      d += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(d), 0xB1, 0xf, 0xf, true));   // lane ^ 1
      d += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(d), 0x4E, 0xf, 0xf, true));   // lane ^ 2
      if ((t & 3) == 0) ndl_s[r0 + 64 * v + (t >> 2)] = -d;
    }
  }
#pragma unroll
  for (int i = 0; i < kAttnTable / 256; ++i) lse_s[t + 256 * i] = t0 + t + 256 * i < n_k ? lv[i] * kLog2e : 1e30f;
}

template <int D, bool KEY>
__device__ __forceinline__ void attn_tiled_body(char* smem, const AttnItem& it, int chunk, int n_k, int h, float scale) {
  using T = AttnTiled<D>;
  float *lse_s = reinterpret_cast<float*>(smem + kAttnRing * T::STAGE), *ndl_s = lse_s + kAttnTable;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int first = chunk * kAttnChunk + wave * 32;         // first token of this wavefront
  const int ns = (n_k + kAttnTile - 1) / kAttnTile, hD = h * D;
  const bool busy = first < n_k;                            // wavefronts without tokens only help with the tiles
  const AttnSwizzled<D> lay(lane);
  AttnStream<D> st(KEY ? it.q : it.q + hD, KEY ? it.g : it.q + 2LL * hD, 3 * hD, KEY ? hD : 3 * hD, n_k, lane, wave);
  st.issue(0, smem, lane, wave);
  if (ns > 1) st.issue(1, smem, lane, wave);
  typename std::conditional<KEY, AttnKeyAcc<D>, AttnQueryAcc<D>>::type acc;
  acc.zero();
  const long long own = min(first + (lane & 31), n_k - 1);
  if constexpr (KEY) {
    acc.from_memory(it.q + own * (3LL * hD) + hD, it.q + own * (3LL * hD) + 2LL * hD, lane);
    attn_make_tables<D, 256 / D>(it, 0, n_k, h, lse_s, ndl_s);
  } else {
    acc.from_memory(it.q + own * (3LL * hD), it.g + own * hD, it.a + own * hD, it.lse + own * h, lane);
  }
  for (int s = 0; s < ns; ++s) {
    wait_async_copies<0>();                                 // tile s, and with it s + 1 (issued one stage ago)
    lds_barrier();                                          // ... everywhere; the ring place of tile s - 1 is free
    if (KEY && s && s % (kAttnTable / kAttnTile) == 0) {
      attn_make_tables<D, D == 128 ? 1 : 2>(it, s * kAttnTile, n_k, h, lse_s, ndl_s);
      lds_barrier();
    }
    if (s + 2 < ns) st.issue(s + 2, smem, lane, wave);
    if (busy) {
      const char* t1 = smem + (s % kAttnRing) * T::STAGE;
      const int rows = min(kAttnTile, n_k - s * kAttnTile), q0 = (s * kAttnTile) % kAttnTable;
      if constexpr (KEY) acc.run(lay, t1, t1 + T::IMG, lse_s + q0, ndl_s + q0, (rows + 31) >> 5, scale, lane);
      else acc.run(lay, t1, t1 + T::IMG, rows, scale, lane);
    }
  }
  lds_barrier();                                            // the tiles have been consumed: the ring becomes the wavefronts' images
  if (busy) {
    char* image = smem + wave * (2 * 32 * (2 * D + 16));
    if constexpr (KEY) {
      attn_store_rows<D>(image, acc.dk, scale, it.o + hD, 3LL * hD, first, n_k, lane);
      attn_store_rows<D>(image + 32 * (2 * D + 16), acc.dv, 1.f, it.o + 2LL * hD, 3LL * hD, first, n_k, lane);
    } else {
      attn_store_rows<D>(image, acc.dq, scale, it.o, 3LL * hD, first, n_k, lane);
    }
  }
}

template <int D>
__global__ void __launch_bounds__(256, D == 128 ? 1 : 3) attn_bwd_tiled_kernel(const uint16_t* __restrict__ qkv, const uint16_t* __restrict__ A,
                                                              const uint16_t* __restrict__ dA, const float* __restrict__ lse,
                                                              int units, int n_k, int h, float scale, int nchunks, uint16_t* __restrict__ dqkv) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  // per XCD a contiguous run of (sample, head, chunk) in the key role (the longer one), then the same run in the query role
  const int per = (units + 7) >> 3, i = blockIdx.x >> 3, unit = (blockIdx.x & 7) * per + (i < per ? i : i - per);
  if (unit >= units) return;
  const int bh = unit / nchunks, c = unit - bh * nchunks, b = bh / h;
  const AttnItem it = attn_item(qkv, A, dA, lse, dqkv, b, bh - b * h, n_k, h, D);
  if (i < per) attn_tiled_body<D, true>(smem, it, c, n_k, h, scale);
  else attn_tiled_body<D, false>(smem, it, c, n_k, h, scale);
}

// ------------------------------------------------------------------------------------------------
// fp32 tensors, d = 32, 64, 128: the same products on v_mfma_f32_32x32x2_f32 (fp32 operands and sums).  A workgroup owns 128
// tokens of one (sample, head) in one of two roles, every wavefront 32 of them: as keys (dK, dV; the queries' rows of q and
// dA stream through LDS in tiles of 32, with their lse and delta) or as queries (dQ; rows of k and v stream).  Layouts (lane
// l, half u = l >> 5): an MFMA takes A[row l & 31][step u] and B[step u][column l & 31]; its result register v is row
// 8 (v >> 2) + 4 u + (v & 3), column l & 31.
//   S, dP: contraction over the head dimension; in a group of 8 dimensions half u multiplies 4 u .. 4 u + 3 (16-byte reads)
//   dV, dK, dQ: contraction over the tile's tokens; step v takes register v of P or dS as B as it is, and A is the tile's
//     element [row of register v][head dimension l & 31]: one 4-byte LDS read per MFMA of 64 cycles, no transpose
// Bound: the matrix cores (fp32 rate), half of a chunk's padding included.  64 samples x 3 heads of 64, 99 kept tokens: 225 us
// with one thread per 16 elements of a token (the plain kernels), 41 us here (18 us of MFMA time if spread evenly; 384
// workgroups of unequal length on 256 CUs).
// ------------------------------------------------------------------------------------------------
typedef float f32x4v_t __attribute__((ext_vector_type(4)));
static constexpr int kAttnF32Tile = 32, kAttnF32Chunk = 128;

template <int D, bool KEY>
struct AttnF32 {
  static constexpr int P = D + 4, CH = D / 4, R = kAttnF32Tile * CH / 256, DB = D / 32;   // LDS pitch, 16-byte pieces per row, per thread
  float own1[D / 2], own2[D / 2];      // k, v (KEY) or q, dA of token l & 31: dimensions 8 c + 4 u .. + 3
  float l, dl;                         // query role: lse and delta of the own token
  f32x16_t acc1[DB], acc2[KEY ? DB : 1];
  f32x4v_t x1[R], x2[R], x3[KEY ? R : 1];
  float xl;

  __device__ __forceinline__ void init(const float* q, const float* a, const float* g, const float* lse, long long ldq, int hd, int h,
                                       int own, int lane) {
    const int u = lane >> 5;
    const float* r1 = q + own * ldq + (KEY ? hd : 0);
    const float* r2 = KEY ? r1 + hd : g + (long long)own * hd;
    float part = 0.f;
#pragma unroll
    for (int c = 0; c < D / 8; ++c) {
      const float4 b1 = *reinterpret_cast<const float4*>(r1 + 8 * c + 4 * u), b2 = *reinterpret_cast<const float4*>(r2 + 8 * c + 4 * u);
      own1[4 * c] = b1.x; own1[4 * c + 1] = b1.y; own1[4 * c + 2] = b1.z; own1[4 * c + 3] = b1.w;
      own2[4 * c] = b2.x; own2[4 * c + 1] = b2.y; own2[4 * c + 2] = b2.z; own2[4 * c + 3] = b2.w;
      if constexpr (!KEY) {
        const float4 o = *reinterpret_cast<const float4*>(a + (long long)own * hd + 8 * c + 4 * u);
        part = fmaf(b2.x, o.x, fmaf(b2.y, o.y, fmaf(b2.z, o.z, fmaf(b2.w, o.w, part))));
      }
    }
    if constexpr (!KEY) { dl = part + __shfl_xor(part, 32); l = lse[(long long)own * h]; }
#pragma unroll
    for (int x = 0; x < DB; ++x)
#pragma unroll
      for (int e = 0; e < 16; ++e) { acc1[x][e] = 0.f; if constexpr (KEY) acc2[x][e] = 0.f; }
  }
  // rows t0 .. t0 + 31 of the other side into registers (past n_k: some valid row, zeroed when stored)
  __device__ __forceinline__ void load(const float* q, const float* a, const float* g, const float* lse, long long ldq, int hd, int h,
                                       int t0, int n_k) {
    const int t = threadIdx.x;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int tok = min(t0 + (t + 256 * r) / CH, n_k - 1), c = 4 * ((t + 256 * r) % CH);
      const float* row = q + tok * ldq + c;
      x1[r] = *reinterpret_cast<const f32x4v_t*>(row + (KEY ? 0 : hd));
      x2[r] = *reinterpret_cast<const f32x4v_t*>(KEY ? g + (long long)tok * hd + c : row + 2 * hd);
      if constexpr (KEY) x3[r] = *reinterpret_cast<const f32x4v_t*>(a + (long long)tok * hd + c);
    }
    if constexpr (KEY) xl = lse[(long long)min(t0 + (t & 31), n_k - 1) * h];
  }
  __device__ __forceinline__ void store_tile(float* s1, float* s2, float* lse_s, float* delta_s, int t0, int n_k) {
    const int t = threadIdx.x;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      asm volatile("" : "+v"(x1[r]), "+v"(x2[r]));         // (loaded registers stay where they are until here)
      if constexpr (KEY) asm volatile("" : "+v"(x3[r]));
      const int row = (t + 256 * r) / CH, ch = (t + 256 * r) % CH;
      const bool ok = t0 + row < n_k;
      f32x4v_t y1 = x1[r], y2 = x2[r];
#pragma unroll
      for (int e = 0; e < 4; ++e) { y1[e] = ok ? y1[e] : 0.f; y2[e] = ok ? y2[e] : 0.f; }
      *reinterpret_cast<f32x4v_t*>(s1 + row * P + 4 * ch) = y1;
      *reinterpret_cast<f32x4v_t*>(s2 + row * P + 4 * ch) = y2;
      if constexpr (KEY) {
        float d = fmaf(y2[0], x3[r][0], fmaf(y2[1], x3[r][1], fmaf(y2[2], x3[r][2], y2[3] * x3[r][3])));
        d = ok ? d : 0.f;
#pragma unroll
        for (int m = 1; m < CH; m <<= 1) d += __shfl_xor(d, m);
        if (ch == 0) delta_s[row] = d;
      }
    }
    if (KEY && t < kAttnF32Tile) lse_s[t] = t0 + t < n_k ? xl : 0.f;
  }
  __device__ __forceinline__ void run(const float* s1, const float* s2, const float* lse_s, const float* delta_s, float scale, int t0,
                                      int n_k, int lane) {
    const int u = lane >> 5, col = lane & 31;
    f32x16_t s, dp;
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] = dp[e] = 0.f;
#pragma unroll
    for (int c = 0; c < D / 8; ++c) {
      const float4 a1 = *reinterpret_cast<const float4*>(s1 + col * P + 8 * c + 4 * u), a2 = *reinterpret_cast<const float4*>(s2 + col * P + 8 * c + 4 * u);
      const float v1[4] = {a1.x, a1.y, a1.z, a1.w}, v2[4] = {a2.x, a2.y, a2.z, a2.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s = __builtin_amdgcn_mfma_f32_32x32x2f32(v1[e], own1[4 * c + e], s, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x2f32(v2[e], own2[4 * c + e], dp, 0, 0, 0);
      }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int r = 8 * (v >> 2) + 4 * u + (v & 3);
      float p = expf(scale * s[v] - (KEY ? lse_s[r] : l));
      if (!KEY) p = t0 + r < n_k ? p : 0.f;                // (KEY: rows past n_k have lse = delta = 0 and zero rows)
      s[v] = p;
      dp[v] = p * (dp[v] - (KEY ? delta_s[r] : dl));
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int off = (8 * (v >> 2) + 4 * u + (v & 3)) * P + col;
#pragma unroll
      for (int x = 0; x < DB; ++x) {
        acc1[x] = __builtin_amdgcn_mfma_f32_32x32x2f32(s1[off + 32 * x], dp[v], acc1[x], 0, 0, 0);          // dK^T or dQ^T
        if constexpr (KEY) acc2[x] = __builtin_amdgcn_mfma_f32_32x32x2f32(s2[off + 32 * x], s[v], acc2[x], 0, 0, 0);   // dV^T
      }
    }
  }
  // out: row 0 of the head's columns in dqkv
  __device__ __forceinline__ void store(float* out, long long ldq, int hd, int own, float scale, int lane) const {
    float* o1 = out + own * ldq + (KEY ? hd : 0) + 4 * (lane >> 5);
#pragma unroll
    for (int x = 0; x < DB; ++x)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        *reinterpret_cast<float4*>(o1 + 32 * x + 8 * q4) =
            make_float4(acc1[x][4 * q4] * scale, acc1[x][4 * q4 + 1] * scale, acc1[x][4 * q4 + 2] * scale, acc1[x][4 * q4 + 3] * scale);
        if constexpr (KEY)
          *reinterpret_cast<float4*>(o1 + hd + 32 * x + 8 * q4) = make_float4(acc2[x][4 * q4], acc2[x][4 * q4 + 1], acc2[x][4 * q4 + 2], acc2[x][4 * q4 + 3]);
      }
  }
};

template <int D, bool KEY>
__device__ __forceinline__ void attn_f32_body(float* smem, const float* qkv, const float* A, const float* dA, const float* lse, int b,
                                              int head, int chunk, int n_k, int h, float scale, float* dqkv) {
  const int t = threadIdx.x, lane = t & 63, hd = h * D;
  const long long row0 = (long long)b * n_k, ldq = 3LL * hd;
  const float *q = qkv + row0 * ldq + head * D, *a = A + row0 * hd + head * D, *g = dA + row0 * hd + head * D, *ls = lse + row0 * h + head;
  float *s1 = smem, *s2 = s1 + kAttnF32Tile * (D + 4), *lse_s = s2 + kAttnF32Tile * (D + 4), *delta_s = lse_s + kAttnF32Tile;
  const int first = chunk * kAttnF32Chunk + (t >> 6) * 32, own = first + (lane & 31);
  const bool busy = first < n_k;                           // wavefronts without tokens only help with the tiles
  AttnF32<D, KEY> f;
  f.init(q, a, g, ls, ldq, hd, h, min(own, n_k - 1), lane);
  f.load(q, a, g, ls, ldq, hd, h, 0, n_k);
  int t0 = 0;
  for (; t0 + kAttnF32Tile < n_k; t0 += kAttnF32Tile) {
    __syncthreads();                                       // the tile before has been consumed
    f.store_tile(s1, s2, lse_s, delta_s, t0, n_k);
    __syncthreads();
    f.load(q, a, g, ls, ldq, hd, h, t0 + kAttnF32Tile, n_k);
    if (busy) f.run(s1, s2, lse_s, delta_s, scale, t0, n_k, lane);
  }
  __syncthreads();
  f.store_tile(s1, s2, lse_s, delta_s, t0, n_k);
  __syncthreads();
  if (busy) f.run(s1, s2, lse_s, delta_s, scale, t0, n_k, lane);
  if (own < n_k) f.store(dqkv + row0 * ldq + head * D, ldq, hd, own, scale, lane);
}

// blockIdx.x: (sample, head, chunk) in the key role, then all of them in the query role (the shorter one)
template <int D>
__global__ void __launch_bounds__(256, D == 128 ? 1 : 2) attn_bwd_f32_kernel(const float* __restrict__ qkv, const float* __restrict__ A,
                                                              const float* __restrict__ dA, const float* __restrict__ lse, int n_units,
                                                              int n_k, int h, float scale, int nchunks, float* __restrict__ dqkv) {
  __shared__ __attribute__((aligned(16))) float smem[2 * kAttnF32Tile * (D + 4) + 2 * kAttnF32Tile];
  const bool key = (int)blockIdx.x < n_units;
  const int unit = key ? blockIdx.x : blockIdx.x - n_units;
  const int chunk = unit % nchunks, bh = unit / nchunks, head = bh % h, b = bh / h;
  if (key) attn_f32_body<D, true>(smem, qkv, A, dA, lse, b, head, chunk, n_k, h, scale, dqkv);
  else attn_f32_body<D, false>(smem, qkv, A, dA, lse, b, head, chunk, n_k, h, scale, dqkv);
}

// ------------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------------
static constexpr size_t kAttnMaxLds = 160 * 1024;

static size_t attn_lds_bytes(int n_k, int d) {
  const int npad = (n_k + 31) & ~31;
  return d == 32 ? AttnLds<32>::bytes(npad) : d == 64 ? AttnLds<64>::bytes(npad) : AttnLds<128>::bytes(npad);
}

// Which kernel runs; decided here alone.  1: one workgroup per (sample, head), 2: tiled, 3: fp32 matrix cores, 0: plain.
// bf16: one workgroup per head where a head is at most two blocks of 32 tokens (64 x 12 heads of 64, one workgroup / tiled: 12.3 /
// 14.0 us at 49 tokens, 7.2 / 10.6 at 25; of 32: 8.6 / 9.9 and 5.2 / 7.8; of 128: 39.9 / 44.3 and 22.9 / 31.9); from three blocks on
// the tiled kernel is ahead (64 x 6 heads: of 64 11.1 / 10.6 at 65 and 16.3 / 14.1 at 99; of 32 8.5 / 8.0 and 11.5 / 9.9; of 128
// 32.4 / 27.5 and 44.2 / 39.1).
// fp32: the matrix-core kernel computes blocks of 32 tokens whatever their number, so the plain one is ahead for heads of a few
// tokens, for the more the wider the head (plain / matrix cores, 1024 x 8 heads: of 32 61 / 76 us at 2 tokens and 97 / 76 at 4; of 64
// 185 / 236 at 4 and 256 / 236 at 6; of 128 652 / 743 at 16 and 802 / 762 at 20) and for fewer where a few heads leave the chip to
// latencies (4 x 4 heads: of 32 5.1 / 5.4 at 1 and 6.1 / 5.5 at 2; of 64 7.6 / 8.1 at 2 and 10.2 / 8.1 at 4; of 128 11.7 / 13.4 at 4
// and 15.0 / 13.4 at 6).
static int few_tokens_f32(int64_t heads, int32_t d) { return heads < 256 ? d / 32 : std::max(2, d * d / 1024); }

static int attention_kernel(int64_t heads, int32_t n_k, int32_t d, int32_t dtype) {
  const int mode = options().attn_mode;                     // explicit overrides (sbp_set_option "attn" = "plain" | "whole" | "tiled")
  if ((d != 32 && d != 64 && d != 128) || mode == 1) return 0;
  // (a grid of the tiled and fp32 kernels, two workgroups of 256 threads per chunk, stays below 2^32 threads)
  const bool grid_fits = heads * ceil_div(n_k, kAttnChunk) < (1 << 23) - 8;
  if (dtype != SBP_BF16) return grid_fits && (mode != 0 || n_k > few_tokens_f32(heads, d)) ? 3 : 0;
  const bool fits = attn_lds_bytes(n_k, d) <= kAttnMaxLds;
  if (mode == 0 ? n_k > 64 : (mode == 3 || !fits)) {
    if (grid_fits) return 2;
  }
  return fits ? 1 : 0;
}
int attention_engine(int32_t n_k, int32_t d, int32_t dtype) { return attention_kernel(4096, n_k, d, dtype); }

template <int D>
static void launch_attn_mfma(const uint16_t* qkv, const uint16_t* A, const uint16_t* dA, const float* lse, int B, int n_k,
                             int h, float scale, uint16_t* dqkv, hipStream_t s) {
  const size_t image = AttnLds<D>::bytes((n_k + 31) & ~31);
  allow_dynamic_lds(reinterpret_cast<const void*>(attn_bwd_mfma_kernel<D>), image);
  SBP_LAUNCH(SBP_PROF_ATTENTION, s, (attn_bwd_mfma_kernel<D>), dim3(h, B), dim3(256), image, s, qkv, A, dA, lse, n_k, h, scale,
             dqkv);
}

template <int D>
static void launch_attn_tiled(const uint16_t* qkv, const uint16_t* A, const uint16_t* dA, const float* lse, int B, int n_k,
                              int h, float scale, uint16_t* dqkv, hipStream_t s) {
  constexpr size_t lds = AttnTiled<D>::LDS;
  allow_dynamic_lds(reinterpret_cast<const void*>(attn_bwd_tiled_kernel<D>), lds);
  const int nchunks = (int)ceil_div(n_k, kAttnChunk), units = B * h * nchunks;
  SBP_LAUNCH(SBP_PROF_ATTENTION, s, (attn_bwd_tiled_kernel<D>), dim3((unsigned)(16 * ceil_div(units, 8))), dim3(256), lds, s, qkv, A, dA,
             lse, units, n_k, h, scale, nchunks, dqkv);
}

template <typename T>
static void launch_attn_plain(const T* qkv, const T* A, const T* dA, const float* lse, int B, int n_k, int h, int d, float scale,
                              T* dqkv, hipStream_t s) {
  const int owners = 256 / (d / 16);
  const dim3 grid((unsigned)ceil_div(n_k, owners), h, B);
  {
    ProfScope scope(SBP_PROF_ATTENTION, s);
    hipLaunchKernelGGL((attn_bwd_plain_kernel<T, 0>), grid, dim3(256), 0, s, qkv, A, dA, lse, n_k, h, d, scale, dqkv);
    hipLaunchKernelGGL((attn_bwd_plain_kernel<T, 1>), grid, dim3(256), 0, s, qkv, A, dA, lse, n_k, h, d, scale, dqkv);
  }
}

template <int D>
static void launch_attn_f32(const float* qkv, const float* A, const float* dA, const float* lse, int B, int n_k, int h, float scale,
                            float* dqkv, hipStream_t s) {
  const int nchunks = (int)ceil_div(n_k, kAttnF32Chunk);
  const long long units = (long long)B * h * nchunks;
  SBP_LAUNCH(SBP_PROF_ATTENTION, s, (attn_bwd_f32_kernel<D>), dim3((unsigned)(2 * units)), dim3(256), 0, s, qkv, A, dA, lse, (int)units,
             n_k, h, scale, nchunks, dqkv);
}

int32_t launch_backward_attention(const void* qkv, const void* A, const void* dA, const float* lse, int32_t B, int32_t n_k,
                                  int32_t h, int32_t d, float scale, int32_t dtype, void* dqkv, hipStream_t s) {
  const int kernel = attention_kernel((int64_t)B * h, n_k, d, dtype);
  if (kernel == 1 || kernel == 2) {
    const uint16_t* q = (const uint16_t*)qkv; const uint16_t* a = (const uint16_t*)A; const uint16_t* g = (const uint16_t*)dA;
    uint16_t* o = (uint16_t*)dqkv;
    if (kernel == 2) {
      if (d == 32) launch_attn_tiled<32>(q, a, g, lse, B, n_k, h, scale, o, s);
      else if (d == 64) launch_attn_tiled<64>(q, a, g, lse, B, n_k, h, scale, o, s);
      else launch_attn_tiled<128>(q, a, g, lse, B, n_k, h, scale, o, s);
    } else {
      if (d == 32) launch_attn_mfma<32>(q, a, g, lse, B, n_k, h, scale, o, s);
      else if (d == 64) launch_attn_mfma<64>(q, a, g, lse, B, n_k, h, scale, o, s);
      else launch_attn_mfma<128>(q, a, g, lse, B, n_k, h, scale, o, s);
    }
  } else if (kernel == 3) {
    const float *q = (const float*)qkv, *a = (const float*)A, *g = (const float*)dA;
    if (d == 32) launch_attn_f32<32>(q, a, g, lse, B, n_k, h, scale, (float*)dqkv, s);
    else if (d == 64) launch_attn_f32<64>(q, a, g, lse, B, n_k, h, scale, (float*)dqkv, s);
    else launch_attn_f32<128>(q, a, g, lse, B, n_k, h, scale, (float*)dqkv, s);
  } else if (dtype == SBP_BF16) {
    launch_attn_plain<uint16_t>((const uint16_t*)qkv, (const uint16_t*)A, (const uint16_t*)dA, lse, B, n_k, h, d, scale,
                                (uint16_t*)dqkv, s);
  } else {
    launch_attn_plain<float>((const float*)qkv, (const float*)A, (const float*)dA, lse, B, n_k, h, d, scale, (float*)dqkv, s);
  }
  return check_launch("backward_attention");
}

}  // namespace sbp
