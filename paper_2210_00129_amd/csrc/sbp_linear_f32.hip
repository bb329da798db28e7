// SBP linear backward for what the bf16 engines do not take: fp32 tensors, and bf16 tensors whose channel counts or
// addresses are not multiples of 8 elements (widened to fp32 on the way into LDS: the products of two bf16 are exact
// there).  Both contractions
//   dX tile:  C[j, i] = sum_o dY[row(j), o] W[o, i]          (rows j = kept rows)
//   dW tile:  C[o, i] = sum_j dY[row(j), o] X_k[j, i]        (j = kept rows of one split)
// run on v_mfma_f32_32x32x2_f32 (fp32 products and sums: 157 TFLOP/s on the chip, twice the vector ALU without packed
// instructions), in one launch per layer together with the column sums for db and the zero fill of the dropped rows.
//
// A workgroup of 4 wavefronts (2 x 2, one 32 x 32 accumulator each) owns a 64 x 64 tile and walks the contraction in stages
// of 64: the next stage is loaded into registers while the current one, in LDS, is multiplied; four workgroups per CU hide
// each other's barriers (128 x 128 tiles, two per CU, were no faster on large layers and worse on small ones).  Both
// operands lie in LDS as [row or column][64 contraction steps] and are read 16 bytes at a time; operands whose contraction
// index is the slow axis in memory (dY and X_k in dW, W in dX) are loaded in blocks of 4 steps x 4 columns per thread and
// written as 4 columns x 4 steps: the transpose is a choice of registers.  Pitch 68 words plus 4 after every fourth row,
// so that 8 neighbouring rows (reads) and rows 4 apart (writes) start on distinct banks (counters: half of the LDS cycles are
// conflicts all the same), and every access of a lane is a fixed offset from one address.  The loop is straight-line code - the partial last stage is
// peeled, gathered and plain rows are different loops - because the compiler copies loaded registers where paths join, and
// the copy waits for the load it was meant to overlap (57 -> 50 us on the layer below).  In a group of 8 contraction steps
// lane half h multiplies steps 4 h .. 4 h + 3, on both operands alike.
// ViT-Tiny fc1 (6336 kept rows, 192 -> 768, with the reduction): 600 us with one thread per output on the vector ALU, 52 us
// here; 20000 rows, 512 -> 512: 198 us = 106 TFLOP/s, with the matrix cores busy 74 % of the cycles of a CU (70 % on fc1).
#include <algorithm>

#include "sbp_internal.h"
#include "sbp_mfma_gemm.h"

namespace sbp {

static constexpr int F32_BT = 64, F32_KB = 64, F32_PITCH = F32_KB + 4;      // tile edge, contraction steps per stage, LDS pitch in words

struct F32Args {
  const void* dY; const int32_t* idx_in; const int32_t* idx_out; const int32_t* idx; const int32_t* inv;
  const void* Xk; const void* W; void* dX;
  float* part; float* dbp;             // [splits][Cout][Cin], [splits][Cout] (dW and db themselves with one split)
  int K, M, Cin, Cout, rows_per_split, splits;
  int chain;                           // rows of a chain of the dW sums (a power of two, at least a stage)
  int n_dx, n_dw, n_db, n_zero;        // workgroups of every kind; in the grid dW and dX units (dx_first: dX units first), column
                                       // sums, zero fill
  int dx_first;
};

// Four elements of T as they come from memory (one vector or four single loads), widened to fp32 when they are used.
// pin() keeps the loaded registers as they are up to that point: without it the compiler moves them to where the LDS
// writes want them right behind the load, and waits for it there.
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
template <typename T, bool VEC> struct F32Quad;
template <> struct F32Quad<float, true> {
  f32x4_t r;
  __device__ __forceinline__ void ld(const float* p) { r = *reinterpret_cast<const f32x4_t*>(p); }
  __device__ __forceinline__ void pin() { asm volatile("" : "+v"(r)); }
  __device__ __forceinline__ void widen(float (&v)[4]) const { v[0] = r[0]; v[1] = r[1]; v[2] = r[2]; v[3] = r[3]; }
  static __device__ __forceinline__ void zero(float* p) { *reinterpret_cast<float4*>(p) = make_float4(0, 0, 0, 0); }
};
template <> struct F32Quad<uint16_t, true> {
  u32x2_t r;
  __device__ __forceinline__ void ld(const uint16_t* p) { r = *reinterpret_cast<const u32x2_t*>(p); }
  __device__ __forceinline__ void pin() { asm volatile("" : "+v"(r)); }
  __device__ __forceinline__ void widen(float (&v)[4]) const { v[0] = bf16_lo(r[0]); v[1] = bf16_hi(r[0]); v[2] = bf16_lo(r[1]); v[3] = bf16_hi(r[1]); }
  static __device__ __forceinline__ void zero(uint16_t* p) { *reinterpret_cast<uint2*>(p) = make_uint2(0, 0); }
};
template <> struct F32Quad<float, false> {
  float r[4];
  __device__ __forceinline__ void pin() { asm volatile("" : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3])); }
  __device__ __forceinline__ void widen(float (&v)[4]) const { v[0] = r[0]; v[1] = r[1]; v[2] = r[2]; v[3] = r[3]; }
};
template <> struct F32Quad<uint16_t, false> {
  uint32_t r[4];
  __device__ __forceinline__ void pin() { asm volatile("" : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3])); }
  __device__ __forceinline__ void widen(float (&v)[4]) const {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = __uint_as_float(r[e] << 16);
  }
};
__device__ __forceinline__ float f32_load(const float* p) { return *p; }
__device__ __forceinline__ float f32_load(const uint16_t* p) { return __uint_as_float((uint32_t)*p << 16); }
__device__ __forceinline__ void f32_store(float* p, float v) { *p = v; }
__device__ __forceinline__ void f32_store(uint16_t* p, float v) { *p = (uint16_t)(bf16_pack(v, 0.f) & 0xffffu); }

// word of contraction steps 4 q .. of tile row r
__device__ __forceinline__ int f32_place(int r, int q) { return r * F32_PITCH + (r >> 2) * 4 + q * 4; }

// Operand whose contraction index is the slow axis: rows k of src, 64 columns from col0.  A thread owns columns cp .. cp + 3
// and steps kr .. kr + 3 of every stage.  Rows past kend are zeroed on the way into LDS (not where they are loaded: that
// would wait for the loads right there); columns past ncols hold other columns, whose results are never stored.  It can
// also add up its columns (db).
template <typename T, bool VEC, bool GATHER>
struct F32SlowLoader {
  const T* src[VEC ? 1 : 4]; const int32_t* idx;
  long long ld;
  int kend, kr, cp;
  int id[4];                            // source rows of the next load
  F32Quad<T, VEC> q[4];                 // [step]: four columns
  float sum[4];

  __device__ __forceinline__ void init(const T* src_, const int32_t* idx_, long long ld_, int col0, int ncols, int k0, int kend_) {
    const int t = threadIdx.x;
    idx = idx_; ld = ld_; kend = kend_;
    cp = (t & 15) * 4; kr = (t >> 4) * 4;
    if constexpr (VEC) src[0] = src_ + min(col0 + cp, ncols - 4);
    else {
#pragma unroll
      for (int e = 0; e < 4; ++e) src[e] = src_ + min(col0 + cp + e, ncols - 1);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) sum[e] = 0.f;
    ids(k0);
  }
  __device__ __forceinline__ void ids(int kbase) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = min(kbase + kr + i, kend - 1);
      id[i] = GATHER ? idx[k] : k;
    }
  }
  __device__ __forceinline__ void load(int kbase) {       // the stage at kbase; then the ids of the one behind it
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (VEC) q[i].ld(src[0] + (long long)id[i] * ld);
      else {
#pragma unroll
        for (int e = 0; e < 4; ++e) q[i].r[e] = src[e][(long long)id[i] * ld];
      }
    }
    ids(kbase + F32_KB);
  }
  template <bool TAIL, bool CS>
  __device__ __forceinline__ void store(float* tile, int kbase) {
    float v[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      q[i].pin();
      q[i].widen(v[i]);
      if constexpr (TAIL) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[i][e] = kbase + kr + i < kend ? v[i][e] : 0.f;
      }
      if constexpr (CS) {
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] += v[i][e];
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      *reinterpret_cast<float4*>(tile + f32_place(cp, kr >> 2) + e * F32_PITCH) = make_float4(v[0][e], v[1][e], v[2][e], v[3][e]);
  }
};

// Operand whose contraction index is contiguous (dY in dX): 64 rows; a thread owns 4 steps of every 16th row.
template <typename T, bool VEC>
struct F32RowLoader {
  const T* rowp[4];
  int kend, kp, r0;
  F32Quad<T, VEC> q[4];

  __device__ __forceinline__ void init(const T* src, const int32_t* idx, long long ld, int row0, int nrows, int kend_) {
    const int t = threadIdx.x;
    kend = kend_;
    kp = (t & 15) * 4; r0 = t >> 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = min(row0 + r0 + 16 * i, nrows - 1);   // rows past the end: computed, never stored
      rowp[i] = src + (idx ? (long long)idx[r] : (long long)r) * ld;
    }
  }
  __device__ __forceinline__ void load(int kbase) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (VEC) q[i].ld(rowp[i] + min(kbase + kp, kend - 4));
      else {
#pragma unroll
        for (int e = 0; e < 4; ++e) q[i].r[e] = rowp[i][min(kbase + kp + e, kend - 1)];
      }
    }
  }
  template <bool TAIL, bool CS>
  __device__ __forceinline__ void store(float* tile, int kbase) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float v[4];
      q[i].pin();
      q[i].widen(v);
      if constexpr (TAIL) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = kbase + kp + e < kend ? v[e] : 0.f;
      }
      *reinterpret_cast<float4*>(tile + f32_place(r0, kp >> 2) + i * (16 * F32_PITCH + 16)) = make_float4(v[0], v[1], v[2], v[3]);
    }
  }
};

static constexpr int F32_TILE_WORDS = F32_BT * F32_PITCH + F32_BT;

// one stage out of LDS; the operands of a group are read while the group before is multiplied (and not earlier: left
// alone, the compiler reads the whole stage first and spills)
// (PART: only the first groups of 8 steps, for the last stage of a contraction, which may be all there is)
template <bool PART = false>
__device__ __forceinline__ void f32_multiply(const float* smem, int wm, int wn, int lane, f32x16_t& acc, int groups = F32_KB / 8) {
  const float* pa = smem + f32_place(wm + (lane & 31), lane >> 5);
  const float* pb = smem + F32_TILE_WORDS + f32_place(wn + (lane & 31), lane >> 5);
  float4 a[2], b[2];
  a[0] = *reinterpret_cast<const float4*>(pa);
  b[0] = *reinterpret_cast<const float4*>(pb);
#pragma unroll
  for (int g = 0; g < F32_KB / 8; ++g) {
    if (PART && g >= groups) break;
    if (g + 1 < F32_KB / 8) {
      a[(g + 1) & 1] = *reinterpret_cast<const float4*>(pa + 8 * (g + 1));
      b[(g + 1) & 1] = *reinterpret_cast<const float4*>(pb + 8 * (g + 1));
    }
    __builtin_amdgcn_sched_barrier(0);
    const float4 x = a[g & 1], y = b[g & 1];
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.x, y.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.y, y.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.z, y.z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.w, y.w, acc, 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Sums over many kept rows are taken in chains that are added up apart, so that the error of a dW element stays about that of one
// chain however long the split is.  FOLD 0: a split of at most 256 rows, one chain; 1: up to 16384 rows, chains of 256 or, from
// 2048 rows on, 128; 2: longer ones, chains of 256 added with the rounding error of every addition carried along (Kahan), which
// takes 16 registers more and would cost thin layers, whose few units wait for their own latencies, 8 % (24.1 -> 26.0 us at 33600
// rows of 60 x 64; 23.2 with plain additions).  2-norm against 64 bits, one running sum / in chains: 5.1e-7 / 2.9e-7 at 6336 rows
// of 768 x 768 (splits of 832), 1.4e-6 / 2.4e-7 at 12608 of 768 x 3072 (6336), 1.6e-6 / 2.6e-7 at 65536 of 768 x 768 (8192).
static constexpr int F32_ONE_CHAIN = 256, F32_PLAIN_FOLD = 16384;

__device__ __forceinline__ void f32_kahan(float& chain, float& total, float& err) {
  const float y = chain - err, t = total + y;
  err = (t - total) - y;
  total = t;
  chain = 0.f;
}

// Stage loop: registers -> LDS -> MFMA (addresses are clamped, so the loads ahead need no bounds check).  CS: operand A
// also sums its columns.
template <bool CS, int FOLD, class LA, class LB>
__device__ __forceinline__ void f32_stage_loop(float* smem, LA& la, LB& lb, int k0, int kend, int chain, int wm, int wn, f32x16_t& acc) {
  const int lane = threadIdx.x & 63;
  float tot[16], err[16];
  float4* ctot = reinterpret_cast<float4*>(smem + 2 * F32_TILE_WORDS) + threadIdx.x;   // (the column sums' chains in LDS: registers are short)
  if constexpr (FOLD != 0) {
#pragma unroll
    for (int v = 0; v < 16; ++v) tot[v] = err[v] = 0.f;
    if constexpr (CS) *ctot = make_float4(0, 0, 0, 0);
  }
  auto fold = [&] {
    if constexpr (FOLD != 0) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        float a = acc[v];
        if (FOLD == 2) f32_kahan(a, tot[v], err[v]);
        else { tot[v] += a; a = 0.f; }
        acc[v] = a;
      }
      if constexpr (CS) {
        const float4 c = *ctot;
        *ctot = make_float4(c.x + la.sum[0], c.y + la.sum[1], c.z + la.sum[2], c.w + la.sum[3]);
#pragma unroll
        for (int e = 0; e < 4; ++e) la.sum[e] = 0.f;
      }
    }
  };
  la.load(k0); lb.load(k0);
  int kb = k0;
  for (; kb + F32_KB < kend; kb += F32_KB) {
    __syncthreads();                                      // everyone has read the stage before
    la.template store<false, CS>(smem, kb);
    lb.template store<false, false>(smem + F32_TILE_WORDS, kb);
    __syncthreads();
    la.load(kb + F32_KB); lb.load(kb + F32_KB);
    f32_multiply(smem, wm, wn, lane, acc);
    if (FOLD != 0 && ((kb - k0 + F32_KB) & (chain - 1)) == 0) fold();
  }
  __syncthreads();
  la.template store<true, CS>(smem, kb);
  lb.template store<true, false>(smem + F32_TILE_WORDS, kb);
  __syncthreads();
  f32_multiply<true>(smem, wm, wn, lane, acc, (kend - kb + 7) >> 3);
  if constexpr (FOLD != 0) {
    fold();
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = tot[v];
    if constexpr (CS) { la.sum[0] = ctot->x; la.sum[1] = ctot->y; la.sum[2] = ctot->z; la.sum[3] = ctot->w; }
  }
}

// dW tile over the kept rows [j0, j1): with sums, smem[64 * step lane + column] holds partial column sums afterwards
template <typename T, bool VEC, bool GATHER, int FOLD>
__device__ __forceinline__ void f32_dw(const F32Args& a, float* smem, int m0, int n0, int j0, int j1, int wm, int wn, bool sums,
                                       f32x16_t& acc) {
  F32SlowLoader<T, VEC, GATHER> la;
  F32SlowLoader<T, VEC, false> lb;
  la.init(static_cast<const T*>(a.dY), a.idx_in, a.Cout, m0, a.Cout, j0, j1);
  lb.init(static_cast<const T*>(a.Xk), nullptr, a.Cin, n0, a.Cin, j0, j1);
  if (!sums) { f32_stage_loop<false, FOLD>(smem, la, lb, j0, j1, a.chain, wm, wn, acc); return; }
  f32_stage_loop<true, FOLD>(smem, la, lb, j0, j1, a.chain, wm, wn, acc);
  __syncthreads();
  *reinterpret_cast<float4*>(smem + (threadIdx.x >> 4) * F32_BT + (threadIdx.x & 15) * 4) = make_float4(la.sum[0], la.sum[1], la.sum[2], la.sum[3]);
  __syncthreads();
}

// One workgroup's unit.  VEC: channel counts and addresses allow 4-element pieces.  FOLD: as above, for the dW
// splits.  Single elements, whose addresses take the most registers, are then faster with three workgroups per CU than spilling
// with four (240 / 287 us at 6336 rows of 769 x 771 in bf16), but not without the chains' sums (69 / 64 us for the dX alone of
// 100000 rows of 65 x 67).
template <typename T, bool VEC, int FOLD>
__global__ void __launch_bounds__(NTHREADS, FOLD && !VEC ? 3 : 4) linear_f32_kernel(const F32Args a) {
  __shared__ __attribute__((aligned(16))) float smem[2 * F32_TILE_WORDS + (FOLD ? 4 * NTHREADS : 0)];
  constexpr int BT = F32_BT;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  const int tiles_n = (a.Cin + BT - 1) / BT;
  const T* dY = static_cast<const T*>(a.dY);
  int wg = blockIdx.x;
  if (a.dx_first) {                                         // (both are multiples of 8: the XCD of a workgroup stays wg & 7)
    if (wg < a.n_dx) wg += a.n_dw;
    else if (wg < a.n_dx + a.n_dw) wg -= a.n_dx;
  }
  f32x16_t acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  const int c = wn + (lane & 31), r4 = wm + 4 * (lane >> 5);    // accumulator v: tile row r4 + 8 (v >> 2) + (v & 3), column c
  if (wg < a.n_dw) {                                        // ---- dW tile of one split
    const int tiles_w = ((a.Cout + BT - 1) / BT) * tiles_n, ntiles = tiles_w * a.splits;
    const int L = (wg & 7) * (a.n_dw >> 3) + (wg >> 3);     // contiguous runs of tiles per XCD (n_dw is a multiple of 8)
    if (L >= ntiles) return;
    const int split = L / tiles_w, rem = L - split * tiles_w;
    const int m0 = (rem / tiles_n) * BT, n0 = (rem % tiles_n) * BT;
    const int j0 = split * a.rows_per_split, j1 = min(a.K, j0 + a.rows_per_split);
    const bool sums = a.dbp && n0 == 0;                     // the first tile column also sums the columns of its dY panel
    if (j0 < j1) {
      if (a.idx_in) f32_dw<T, VEC, true, FOLD>(a, smem, m0, n0, j0, j1, wm, wn, sums, acc);
      else f32_dw<T, VEC, false, FOLD>(a, smem, m0, n0, j0, j1, wm, wn, sums, acc);
    }
    float* part = a.part + (long long)split * a.Cout * a.Cin;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int o = m0 + r4 + 8 * (v >> 2) + (v & 3);
      if (o < a.Cout && n0 + c < a.Cin) part[(long long)o * a.Cin + n0 + c] = acc[v];
    }
    if (sums && t < BT && m0 + t < a.Cout) {                // the 16 step lanes of a column added in a fixed order
      float s = 0.f;
      if (j0 < j1)
        for (int r = 0; r < 16; ++r) s += smem[r * BT + t];
      a.dbp[(long long)split * a.Cout + m0 + t] = s;
    }
    return;
  }
  wg -= a.n_dw;
  if (wg < a.n_dx) {                                        // ---- dX tile
    const int ntiles = ((a.K + BT - 1) / BT) * tiles_n;
    const int L = (wg & 7) * (a.n_dx >> 3) + (wg >> 3);
    if (L >= ntiles) return;
    const int m0 = (L / tiles_n) * BT, n0 = (L % tiles_n) * BT;
    F32RowLoader<T, VEC> la;
    F32SlowLoader<T, VEC, false> lb;
    la.init(dY, a.idx_in, a.Cout, m0, a.K, a.Cout);
    lb.init(static_cast<const T*>(a.W), nullptr, a.Cin, n0, a.Cin, 0, a.Cout);
    f32_stage_loop<false, 0>(smem, la, lb, 0, a.Cout, 0, wm, wn, acc);
    int* ids = reinterpret_cast<int*>(smem);
    __syncthreads();
    if (t < BT) { const int j = min(m0 + t, a.K - 1); ids[t] = a.idx_out ? a.idx_out[j] : j; }
    __syncthreads();
    T* dX = static_cast<T*>(a.dX);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int r = r4 + 8 * (v >> 2) + (v & 3);
      if (m0 + r < a.K && n0 + c < a.Cin) f32_store(dX + (long long)ids[r] * a.Cin + n0 + c, acc[v]);
    }
    return;
  }
  wg -= a.n_dx;
  if (wg < a.n_db) {                                        // ---- db without dW: 64 columns over one split's rows
    const int chunks = (a.Cout + 63) / 64, split = wg / chunks, c = (wg % chunks) * 64 + lane;
    const int j0 = split * a.rows_per_split, j1 = min(a.K, j0 + a.rows_per_split);
    float s = 0.f, err = 0.f;
    if (c < a.Cout) {
      for (int jc = j0; jc < j1; jc += F32_ONE_CHAIN) {
        float q = 0.f;
#pragma unroll 4
        for (int j = jc + wave; j < min(j1, jc + F32_ONE_CHAIN); j += 4) q += f32_load(dY + (long long)(a.idx_in ? a.idx_in[j] : j) * a.Cout + c);
        f32_kahan(q, s, err);
      }
    }
    smem[t] = s;
    __syncthreads();
    if (t < 64 && c < a.Cout) a.dbp[(long long)split * a.Cout + c] = ((smem[t] + smem[64 + t]) + smem[128 + t]) + smem[192 + t];
    return;
  }
  wg -= a.n_db;
  T* dX = static_cast<T*>(a.dX);                            // ---- zero fill: a wavefront looks 64 rows up at once
  constexpr int V = VEC ? 4 : 1;
  const int pieces = a.Cin / V;
  for (uint32_t base = (wg * 4 + wave) * 64; base < (uint32_t)a.M; base += a.n_zero * 256) {   // (unsigned: M may be the largest int)
    const uint32_t m = base + lane;
    bool dropped = false;
    if (m < (uint32_t)a.M) {
      const int j = a.inv[m];
      dropped = !((unsigned)j < (unsigned)a.K && a.idx[j] == (int)m);
    }
    unsigned long long mask = __ballot(dropped);
    T* rows = dX + (long long)base * a.Cin;
    if (pieces < 64 && pieces <= __popcll(mask)) {           // narrow rows: the pieces of the 64 rows side by side over the lanes
      const uint32_t magic = (1u << 20) / pieces + 1;       // e / pieces = e magic >> 20 for e < 64 pieces
      for (uint32_t e = lane; e < 64u * pieces; e += 64)
        if ((mask >> ((e * magic) >> 20)) & 1) {
          if constexpr (VEC) F32Quad<T, true>::zero(rows + e * V);
          else rows[e] = (T)0;
        }
      continue;
    }
    while (mask) {
      const int b = __ffsll((long long)mask) - 1;
      mask &= mask - 1;
      T* row = rows + (long long)b * a.Cin;
      for (int p = lane; p < pieces; p += 64) {
        if constexpr (VEC) F32Quad<T, true>::zero(row + p * V);
        else row[p] = (T)0;
      }
    }
  }
}

// dW splits of a layer.  The rows are cut so that a dW unit is about as long as half an even share of the whole work (four
// workgroups per CU), at least 256 rows; a single split writes dW and db itself, which saves the reduction launch.
void plan_linear_f32(int64_t K, int32_t Cin, int32_t Cout, int* splits, int* rows_per_split) {
  const int64_t tiles_n = ceil_div(Cin, F32_BT), tiles_w = ceil_div(Cout, F32_BT) * tiles_n;
  const int64_t steps = ceil_div(K, F32_BT) * tiles_n * Cout + tiles_w * K;   // of all units
  const int64_t rows = std::max<int64_t>(256, ceil_div(steps, 2 * 4 * 256));
  const int64_t n = std::min<int64_t>(64, std::max<int64_t>(1, ceil_div(K, rows)));
  *rows_per_split = (int)(ceil_div(ceil_div(K, n), F32_KB) * F32_KB);
  *splits = (int)ceil_div(K, *rows_per_split);
}

template <typename T, bool VEC>
static auto f32_kernel(int fold) {
  return fold == 0 ? linear_f32_kernel<T, VEC, 0> : (fold == 1 ? linear_f32_kernel<T, VEC, 1> : linear_f32_kernel<T, VEC, 2>);
}

void launch_linear_f32(int splits, int rows_per_split, const void* dY, const int32_t* idx_in, const int32_t* idx_out,
                       const int32_t* idx, const int32_t* inv, const void* Xk, const void* W, int64_t M, int64_t K, int32_t Cin,
                       int32_t Cout, int32_t dtype, bool want_dw, float* part, float* dbp, void* dX, hipStream_t s) {
  F32Args a{};
  a.dY = dY; a.idx_in = idx_in; a.idx_out = idx_out; a.idx = idx; a.inv = inv; a.Xk = Xk; a.W = W; a.dX = dX;
  a.part = part; a.dbp = dbp;
  a.K = (int)K; a.M = (int)M; a.Cin = Cin; a.Cout = Cout; a.rows_per_split = rows_per_split; a.splits = splits;
  const int64_t tiles_n = ceil_div(Cin, F32_BT);
  if (want_dw) a.n_dw = (int)(8 * ceil_div(ceil_div(Cout, F32_BT) * tiles_n * splits, 8));
  else if (dbp) a.n_db = (int)(ceil_div(Cout, 64) * splits);
  if (dX) a.n_dx = (int)(8 * ceil_div(ceil_div(K, F32_BT) * tiles_n, 8));
  a.dx_first = Cout > rows_per_split;                       // the longer kind first: a late long unit would run on alone
  if (dX && idx_out && M > K) a.n_zero = (int)std::min<int64_t>(256, ceil_div(M, 256));
  const unsigned grid = (unsigned)(a.n_dw + a.n_dx + a.n_db + a.n_zero);
  if (grid == 0) return;
  const uintptr_t addr = (uintptr_t)dY | (uintptr_t)(want_dw ? Xk : nullptr) | (uintptr_t)(dX ? W : nullptr) | (uintptr_t)dX;
  const bool f32 = dtype == SBP_F32, vec = Cin % 4 == 0 && Cout % 4 == 0 && addr % (f32 ? 16 : 8) == 0;
  a.chain = rows_per_split > 2048 && rows_per_split <= F32_PLAIN_FOLD ? 128 : 256;
  const int fold = !want_dw || rows_per_split <= F32_ONE_CHAIN ? 0 : (rows_per_split <= F32_PLAIN_FOLD ? 1 : 2);
  auto kernel = f32 ? (vec ? f32_kernel<float, true>(fold) : f32_kernel<float, false>(fold))
                    : (vec ? f32_kernel<uint16_t, true>(fold) : f32_kernel<uint16_t, false>(fold));
  SBP_LAUNCH(SBP_PROF_DW_GEMM, s, kernel, dim3(grid), dim3(NTHREADS), 0, s, a);
}

}  // namespace sbp
