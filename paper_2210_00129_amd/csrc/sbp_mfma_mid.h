// The 128-wide engine for the two bf16 contractions of the SBP linear backward (paper, eq:backward_fc_sbp): layers that do
// not fill the chip with 256-wide tiles (sbp_mfma_big.h), any channel counts that are multiples of 8, any offsets.
//
// A workgroup of 4 wavefronts owns a 128 x 128 tile (dX also 64 x 128), 64 x 64 (32 x 64) per wavefront, and walks the
// contraction in stages of 32 through a ring of four LDS stages of 16 KB.  Such layers are a few hundred workgroups of 10 to
// 130 stages, one or two per CU, so a launch is as long as one workgroup's chain of stages, and what bounds it is the time a
// wavefront that is nearly alone on its SIMD takes to issue a stage (MFMAs of 256 cycles, 12 to 18 LDS reads, 4 copies):
//   * the fragments of a step (16 deep, 4 MFMAs) are read from LDS between the MFMAs of the step before (two sets of
//     registers, order fixed by half_order), so nothing waits out an LDS round trip and the matrix core runs while reads issue;
//   * the copies of three stages are in flight (global -> LDS, counted with vmcnt); one barrier per stage, which waits for no
//     LDS reads (ring_loop);
//   * db comes out of the dW units: v_dot2 against ones on the dY fragments in registers, the unit (split, tile row, tile
//     column) with tile column = split mod columns sums its panel.  (As workgroups of their own the sums read dY_k a third time.)
// dX alone, warm, a call: 60 rows of 384 -> 1536 (48 stages) 16.3 us with stages of 64 in a ring of two and all reads of a step
// ahead of its MFMAs, now 10.2; 4200 rows of 512 -> 2048 24.2 -> 20.1.  dW alone of 4200 x 512 -> 2048 29.8 -> 22.4 (also for fewer
// splits).  32768 rows of 2048 x 2048: 737 -> 790 TFLOP/s (the large tiles 1113).  Rings of 5 and 8 stages with one workgroup per CU
// and of 3 with three were slower (60 rows: 15.9, 17.0, 15.9 against 14.4 us for the whole call): latency of memory is not the bound.
// LDS tile layouts and swizzles are those of sbp_mfma_gemm.h.
#ifndef SBP_MFMA_MID_H_
#define SBP_MFMA_MID_H_

#include <type_traits>

#include "sbp_mfma_gemm.h"

namespace sbp {
namespace mid {

static constexpr int BT = 128, KB = 32, NS = 4;
static constexpr int TILE = BT * KB * 2;            // bytes of a 128-wide operand tile of a stage
static constexpr int RING = NS * 2 * TILE;

// FIRST: the first step of a chain of sums (starts from 0 instead of acc)
template <bool SWAP, int FM, bool FIRST = false>
__device__ __forceinline__ void mfma_step(f32x16_t (&acc)[FM][2], const bf16x8_t (&a)[FM], const bf16x8_t (&b)[2]) {
  const f32x16_t zero = {};
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const f32x16_t c = FIRST ? zero : acc[i][j];
      acc[i][j] = SWAP ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j], a[i], c, 0, 0, 0)
                       : __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], c, 0, 0, 0);
    }
}
template <int FM>
__device__ __forceinline__ void add_acc(f32x16_t (&sum)[FM][2], const f32x16_t (&acc)[FM][2]) {
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) sum[i][j] += acc[i][j];
}

// at most n stages of CPS copies still under way (wave-uniform; more than N count as N)
template <int CPS, int N = NS - 2>
__device__ __forceinline__ void wait_stages(int n) {
  if (n >= N) wait_async_copies<N * CPS>();
  else if constexpr (N > 0) wait_stages<CPS, N - 1>(n);
}

// Instruction order of half a stage, given to the scheduler as groups (the code of the half is written before the call): NM
// MFMAs, the LDS reads behind the first of them, then the copies (the compiler keeps LDS reads and copies in the order in which
// they are written).  A wavefront issues in order: reads ahead of the MFMAs would leave the matrix core idle while they issue.
template <int MASK, int N>
__device__ __forceinline__ void sched_group() {
  if constexpr (N > 0) __builtin_amdgcn_sched_group_barrier(MASK, N, 0);
}
template <int NM, int NREAD, int NCOPY, int I = 0>
__device__ __forceinline__ void half_order() {
  constexpr int RS = NM > 2 ? NM - 1 : 1, PER = (NREAD + RS - 1) / RS;     // slots that carry reads, reads of a slot
  constexpr int CS = NM - RS + 1, c = I - (RS - 1);                        // slots that carry copies, number of this one
  sched_group<0x008, 1>();
  if constexpr (I < RS) sched_group<0x100, (NREAD - PER * I < PER ? NREAD - PER * I : PER)>();
  if constexpr (c >= 0) sched_group<0x010, NCOPY * (c + 1) / CS - NCOPY * c / CS>();
  if constexpr (I + 1 < NM) half_order<NM, NREAD, NCOPY, I + 1>();
}

// The stage ring.  Iteration s consumes stage s in two halves of one 16-deep step.  First half: MFMAs of step 0, step 1's
// fragments are read.  Then the barrier that publishes stage s + 1; every wavefront has the fragments of stage s - 1 in registers
// by then (its MFMAs of step 1 came before), so that buffer is free: second half: MFMAs of step 1, the fragments of stage s + 1,
// step 0, are read, and the copies of stage s + NS - 1 go to the buffer of stage s - 1.  The barrier waits for no LDS reads.
// P::CHAIN (dW): the sums run in chains of that many stages, each from 0, that are added up apart - the splits are as long as the
// schedule wants them, but one running sum over 900 rows is 1.7e-7 off 64 bits (2-norm) where sums of 320 are 1.0e-7 off.
// P: prefetch(s) - row ids of stage s; issue(buffer, kvalid) - the copies of the next stage, kvalid < 32 in a partial last
// one; read(buffer, step, a, b); extra(a).
template <class P>
__device__ __forceinline__ void ring_loop(char* smem, P& pb, int nk, int kvalid_last, f32x16_t (&acc)[P::FM][2]) {
  constexpr int FM = P::FM, CPS = P::CPS, STAGE = P::STAGE, NM = 2 * FM;
#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < nk) {
      pb.prefetch(s);
      pb.issue(smem + s * STAGE, s == nk - 1 ? kvalid_last : KB);
    }
  wait_stages<CPS>(min(NS - 2, nk - 1));
  lds_barrier();
  bf16x8_t pa[FM], pbf[2], qa[FM], qb[2];
  pb.read(smem, 0, pa, pbf);
  char *cur = smem, *nxt = smem + STAGE, *dst = smem + (NS - 1) * STAGE;
  auto turn = [&] {
    dst = cur;
    cur = nxt;
    nxt = nxt == smem + (NS - 1) * STAGE ? smem : nxt + STAGE;
  };
  f32x16_t sum[FM][2];                               // (only where there are chains)
  int s = 0;
  auto steady = [&](auto first) {
    pb.prefetch(s + NS - 1);
    pb.read(cur, 1, qa, qb);
    mfma_step<P::SWAP, FM, decltype(first)::value>(acc, pa, pbf);
    pb.extra(pa[0]);
    half_order<NM, P::NREAD + P::NPRE, 0>();
    __builtin_amdgcn_sched_barrier(0);
    wait_async_copies<(NS - 3) * CPS>();             // stage s + 1 has landed
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    pb.read(nxt, 0, pa, pbf);
    pb.issue(dst, KB);
    mfma_step<P::SWAP, FM>(acc, qa, qb);
    pb.extra(qa[0]);
    half_order<NM, P::NREAD, CPS>();
    __builtin_amdgcn_sched_barrier(0);
    turn();
    ++s;
  };
  // stage s + NS - 1 exists and is not the last one
  if constexpr (P::CHAIN > 0) {
    zero_acc<FM, 2>(sum);
    while (s + P::CHAIN <= nk - NS) {
      steady(std::true_type{});
      for (int e = s + P::CHAIN - 1; s < e;) steady(std::false_type{});
      add_acc<FM>(sum, acc);
    }
    zero_acc<FM, 2>(acc);                            // the last chain: what is left, up to CHAIN + NS - 1 stages
  }
  while (s < nk - NS) steady(std::false_type{});
  for (; s < nk; ++s) {                              // the same with the end of the operands in view
    const bool more = s + NS - 1 < nk;
    if (more) pb.prefetch(s + NS - 1);
    pb.read(cur, 1, qa, qb);
    mfma_step<P::SWAP, FM>(acc, pa, pbf);
    pb.extra(pa[0]);
    if (s + 1 < nk) {
      wait_stages<CPS, NS - 3>(nk - 2 - s);          // stages s + 2 .. (at most s + NS - 2 have been issued) may be under way
      lds_barrier();
      pb.read(nxt, 0, pa, pbf);
      if (more) pb.issue(dst, s + NS == nk ? kvalid_last : KB);
    }
    mfma_step<P::SWAP, FM>(acc, qa, qb);
    pb.extra(qa[0]);
    turn();
  }
  if constexpr (P::CHAIN > 0) add_acc<FM>(acc, sum);
  lds_barrier();                                     // the ring is free
}

// What the copies of a partial last stage read past the end of an operand: zeros on both sides (zero times an infinite value is NaN).
__device__ const uint4 zeros[1] = {};
__device__ __forceinline__ const char* zero_line() { return reinterpret_cast<const char*>(zeros); }

// ---- copies of a slow tile [32 k][128 columns]: 8 blocks of 4 rows, 2 per wavefront ---------------------------------
struct SlowCopy {
  const char* p[2];       // this lane's piece of block n in the next stage (operands with consecutive rows)
  size_t ld, step;        // bytes of a row, of a stage
  int kl;                 // row within the stage of block 0 (block 1: + 4)
  uint32_t colb;          // column bytes of this lane
  __device__ __forceinline__ void init(const void* src, size_t ld_bytes, int col0, int ncols, int lane, int wave) {
    ld = ld_bytes; step = KB * ld_bytes;
    kl = 8 * wave + (lane >> 4);
    colb = 2u * (uint32_t)min(col0 + 8 * ((lane & 15) ^ (((lane >> 4) & 3) << 2)), ncols - 8);
#pragma unroll
    for (int n = 0; n < 2; ++n) p[n] = static_cast<const char*>(src) + (size_t)(kl + 4 * n) * ld + colb;
  }
  __device__ __forceinline__ void issue(char* tile, int kvalid, int wave) {
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const char* q = kvalid < KB && kl + 4 * n >= kvalid ? zero_line() : p[n];
      async_copy16(q, tile + (2 * wave + n) * 1024);
      p[n] += step;
    }
  }
};

// X_k in groups of 8 rows, [row group][channel][8 rows]: a stage is 4 groups x 128 pieces of 16 bytes, copied as they lie (a
// wavefront copies one group), and a fragment is one 16-byte LDS read per lane instead of two transposing reads.
struct GroupCopy {
  const char* p[2];       // this lane's piece of columns 0 .. 63 and 64 .. 127 in the next stage
  size_t ld, step;        // bytes of a group, of a stage
  __device__ __forceinline__ void init(const void* src, int Cin, int col0, int lane, int wave) {
    ld = (size_t)Cin * 16; step = KB / 8 * ld;
#pragma unroll
    for (int n = 0; n < 2; ++n) p[n] = static_cast<const char*>(src) + (size_t)wave * ld + (size_t)min(col0 + 64 * n + lane, Cin - 1) * 16;
  }
  __device__ __forceinline__ void issue(char* tile, int kvalid, int wave) {
    const bool past = kvalid < KB && 8 * wave >= kvalid;             // (rows past the last one of its group are stored as zeros)
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      async_copy16(past ? zero_line() : p[n], tile + (2 * wave + n) * 1024);
      p[n] += step;
    }
  }
};

// ---- dX = dY_k W -------------------------------------------------------------------------------------------------------
template <int FM_>
struct DxProb {
  static constexpr bool SWAP = true;                 // a lane ends with 4 consecutive input channels of one row
  static constexpr int FM = FM_, CPS = FM + 2, NREAD = FM + 4, NPRE = 0, CHAIN = 0, A_BYTES = 64 * FM * KB * 2, STAGE = A_BYTES + TILE;
  const char* pa[FM];
  SlowCopy cb;
  int wave, kchunk, a_off[2], b_off[2];
  __device__ __forceinline__ void extra(const bf16x8_t&) {}
  __device__ __forceinline__ void prefetch(int) {}
  __device__ __forceinline__ void issue(char* buf, int kvalid) {
#pragma unroll
    for (int n = 0; n < FM; ++n) {
      async_copy16(kvalid < KB && kchunk >= kvalid ? zero_line() : pa[n], buf + (FM * wave + n) * 1024);
      pa[n] += KB * 2;
    }
    cb.issue(buf + A_BYTES, kvalid, wave);
  }
  __device__ __forceinline__ void read(const char* buf, int ks, bf16x8_t (&a)[FM], bf16x8_t (&b)[2]) const {
    read_slow_frags<BT, 2>(buf + A_BYTES, b_off, ks, b);
#pragma unroll
    for (int f = 0; f < FM; ++f) a[f] = *reinterpret_cast<const bf16x8_t*>(buf + a_off[ks] + f * (32 * KB * 2));
  }
};

// BMX kept rows (128 or 64) x 128 input channels
template <int BMX>
__device__ __forceinline__ void dx_tile(char* smem, const uint16_t* __restrict__ dY, const int32_t* __restrict__ idx_in,
                                        const int32_t* __restrict__ idx_out, const uint16_t* __restrict__ W, int K, int Cin,
                                        int Cout, uint16_t* __restrict__ dX, int m0, int n0) {
  constexpr int FM = BMX / 64;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = (wave >> 1) * (BMX / 2), wn = (wave & 1) * 64;
  DxProb<FM> pb;
  pb.wave = wave;
  pb.kchunk = 8 * ((lane & 3) ^ ((lane >> 4) & 3));
#pragma unroll
  for (int n = 0; n < FM; ++n) {
    const int r = min(m0 + 16 * (FM * wave + n) + (lane >> 2), K - 1);
    pb.pa[n] = reinterpret_cast<const char*>(dY + (size_t)(idx_in ? idx_in[r] : r) * Cout + pb.kchunk);
  }
  pb.cb.init(W, (size_t)Cin * 2, n0, Cin, lane, wave);
  {
    const int row = wm + (lane & 31), sw = (lane >> 2) & 3;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) pb.a_off[ks] = row * (KB * 2) + (((2 * ks + (lane >> 5)) ^ sw) << 4);
  }
  slow_tile_lane_offs<BT, 2>(wn, lane, pb.b_off);
  f32x16_t acc[FM][2];
  zero_acc<FM, 2>(acc);
  const int nk = (Cout + KB - 1) / KB;
  ring_loop(smem, pb, nk, Cout - (nk - 1) * KB, acc);

  // epilogue: 64 rows at a time through LDS, whole 16-byte pieces of the (scattered) rows
  constexpr int PITCH = BT * 2 + 16;
  const int pc = t & 15, pr = t >> 4;
  const bool col_ok = n0 + 8 * pc < Cin;
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    char* row = smem + ((wave >> 1) * 32 + (lane & 31)) * PITCH + (wn + 4 * (lane >> 5)) * 2;
#pragma unroll
    for (int jn = 0; jn < 2; ++jn)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<uint2*>(row + (32 * jn + 8 * q) * 2) =
            make_uint2(bf16_pack(acc[i][jn][4 * q + 0], acc[i][jn][4 * q + 1]), bf16_pack(acc[i][jn][4 * q + 2], acc[i][jn][4 * q + 3]));
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int r = pr + 16 * p;                       // staged row: half r >> 5, row r & 31
      const int j = m0 + (r >> 5) * (BMX / 2) + 32 * i + (r & 31);
      if (j < K && col_ok)
        *reinterpret_cast<uint4*>(dX + (long long)(idx_out ? idx_out[j] : j) * Cin + n0 + 8 * pc) =
            *reinterpret_cast<const uint4*>(smem + r * PITCH + pc * 16);
    }
    __syncthreads();
  }
}

// ---- dW partial = dY_k[j0:j1]^T X_k[j0:j1] -----------------------------------------------------------------------------
// The two wavefronts that own the same 64 rows of the tile (and hold the same dY fragments) take them in opposite order, so that
// "the column sums of fragment 0" is every row's sum once.  XT: X_k lies in row groups (j0 is a whole number of them); the same
// products in the same order.
template <bool GATHER, bool DB, bool XT>
struct DwProb {
  static constexpr bool SWAP = false;
  static constexpr int FM = 2, CPS = 4, NREAD = XT ? 6 : 8, NPRE = GATHER ? 1 : 0, CHAIN = 10, STAGE = 2 * TILE;       // (the two row ids are one read)
  SlowCopy ca;
  std::conditional_t<XT, GroupCopy, SlowCopy> cb;
  const char* dY;
  const int* rows;                 // LDS table: row of dY of kept row j0 + i, whole stages
  int rid[2];
  int wave, a_off[2], b_off[2];
  float sum[DB ? 4 : 1];           // one chain per word of a fragment
  __device__ __forceinline__ void extra(const bf16x8_t& a) {
    if constexpr (DB) {
      const bf16x2_t ones = __builtin_bit_cast(bf16x2_t, 0x3f803f80u);
      const uint4 w = __builtin_bit_cast(uint4, a);
      unsigned v[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        asm("" : "+v"(v[q]));       // (otherwise the four words are folded into the first one)
        sum[q] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, v[q]), ones, sum[q], false);
      }
    }
  }
  __device__ __forceinline__ void prefetch(int s) {
    if constexpr (GATHER) {
#pragma unroll
      for (int n = 0; n < 2; ++n) rid[n] = rows[s * KB + ca.kl + 4 * n];
    }
  }
  __device__ __forceinline__ void issue(char* buf, int kvalid) {
    if constexpr (GATHER) {        // (the table repeats the last row past the end)
#pragma unroll
      for (int n = 0; n < 2; ++n)
        async_copy16(kvalid < KB && ca.kl + 4 * n >= kvalid ? zero_line() : dY + (uint64_t)(uint32_t)rid[n] * (uint32_t)ca.ld + ca.colb,
                     buf + (2 * wave + n) * 1024);
    } else {
      ca.issue(buf, kvalid, wave);
    }
    cb.issue(buf + TILE, kvalid, wave);
  }
  __device__ __forceinline__ void read(const char* buf, int ks, bf16x8_t (&a)[2], bf16x8_t (&b)[2]) const {
    if constexpr (XT) {
#pragma unroll
      for (int f = 0; f < 2; ++f) b[f] = *reinterpret_cast<const bf16x8_t*>(buf + TILE + b_off[f] + ks * (2 * BT * 16));
    } else {
      read_slow_frags<BT, 2>(buf + TILE, b_off, ks, b);
    }
    read_slow_frags<BT, 2>(buf, a_off, ks, a);
  }
};

// dbp (DB): the column sums of the tile's dY panel over [j0, j1)
template <bool GATHER, bool DB, bool XT>
__device__ __forceinline__ void dw_tile(char* smem, const uint16_t* __restrict__ dY, const int32_t* __restrict__ idx,
                                        const uint16_t* __restrict__ Xk, int Cin, int Cout, int j0, int j1,
                                        float* __restrict__ part, int m0, int n0, float* __restrict__ dbp) {
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), flip = wave & 1;
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
  const int nrows = j1 - j0, nk = (nrows + KB - 1) / KB;
  DwProb<GATHER, DB, XT> pb;
  pb.wave = wave;
  pb.dY = reinterpret_cast<const char*>(dY);
  pb.ca.init(GATHER ? dY : dY + (size_t)j0 * Cout, (size_t)Cout * 2, m0, Cout, lane, wave);
  if constexpr (XT) pb.cb.init(Xk + (size_t)j0 * Cin, Cin, n0, lane, wave);
  else pb.cb.init(Xk + (size_t)j0 * Cin, (size_t)Cin * 2, n0, Cin, lane, wave);
  pb.rows = nullptr;
  if constexpr (GATHER) {
    int* rows = reinterpret_cast<int*>(smem + RING);
    for (int i = t; i < nk * KB; i += 256) rows[i] = idx[min(j0 + i, j1 - 1)];
    __syncthreads();
    pb.rows = rows;
  }
#pragma unroll
  for (int q = 0; q < (DB ? 4 : 1); ++q) pb.sum[q] = 0.f;
  {
    int off[2];
    slow_tile_lane_offs<BT, 2>(wm, lane, off);
    pb.a_off[0] = flip ? off[1] : off[0];
    pb.a_off[1] = flip ? off[0] : off[1];
  }
  if constexpr (XT) {
#pragma unroll
    for (int f = 0; f < 2; ++f) pb.b_off[f] = ((lane >> 5) * BT + wn + 32 * f + (lane & 31)) * 16;
  } else {
    slow_tile_lane_offs<BT, 2>(wn, lane, pb.b_off);
  }
  f32x16_t acc[2][2];
  zero_acc<2, 2>(acc);
  ring_loop(smem, pb, nk, nrows - (nk - 1) * KB, acc);

  if constexpr (DB) {                // lanes l and l + 32 hold the two j groups of column l % 32 of fragment `flip`
    float s = (pb.sum[0] + pb.sum[1]) + (pb.sum[2] + pb.sum[3]);
    s += __shfl_xor(s, 32);
    const int o = m0 + wm + 32 * flip + (lane & 31);
    if (lane < 32 && o < Cout) dbp[o] = s;
  }
  // register v of lane l of block (i, j) is C[row wm + 32 (i ^ flip) + 8 (v >> 2) + 4 (l >> 5) + (v & 3)][column wn + 32 j + (l & 31)]
  if (m0 + BT <= Cout && n0 + BT <= Cin) {         // interior tile: no bounds checks
    float* p = part + (long long)(m0 + wm + 32 * flip + 4 * (lane >> 5)) * Cin + n0 + wn + (lane & 31);
    const long long other = flip ? -32ll * Cin : 32ll * Cin;          // from fragment 0's rows to fragment 1's
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        float* row = p + i * other + (long long)(8 * (v >> 2) + (v & 3)) * Cin;
        row[0] = acc[i][0][v];
        row[32] = acc[i][1][v];
      }
  } else {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int o = m0 + wm + 32 * (i ^ flip) + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3), c = n0 + wn + (lane & 31);
        float* row = part + (long long)o * Cin + c;
#pragma unroll
        for (int jn = 0; jn < 2; ++jn)
          if (o < Cout && c + 32 * jn < Cin) row[32 * jn] = acc[i][jn][v];
      }
  }
}

// db alone: the column sums of one split, 64 channels from c0 on, in the chains of dw_tile (the same bits whichever outputs are
// wanted).  Thread (x = t & 31, y = t >> 5) owns 2 channels and rows 2 y, 2 y + 1 of every 16: word y & 3 of half y >> 2.  These
// are few workgroups of long chains, so what bounds them is the instructions of a step and the loads in flight: the rows' offsets are
// staged in LDS as they are added to the base (WIDE: tensors of 4 GB and more, row ids), and U steps are loaded at a time with no
// shorter loop behind them, which would wait for every row.  db alone, a call, with a loop over 64-bit addresses / now (operands from
// memory): 900 rows of 1000 channels 6.5 / 5.1 us (9.3 / 6.5), 8400 of 256 9.3 / 7.2 (12.5 / 8.3), 16800 of 1024 14.4 / 9.8 (17.8 / 12.5),
// 33600 of 256 12.7 / 9.3 (17.0 / 11.4), 60000 of 288 16.9 / 12.5 (17.4 / 13.3).
static constexpr int kColumns = 64;
template <bool WIDE>
__device__ __forceinline__ void colsum_block(char* smem, const uint16_t* __restrict__ dY, const int32_t* __restrict__ idx, int Cout,
                                             int j0, int j1, int c0, float* __restrict__ dbp) {
  constexpr int U = 16;
  const int t = threadIdx.x, x = t & 31, y = t >> 5, n = j1 - j0, steps = (n + 15) / 16;
  uint32_t* rows = reinterpret_cast<uint32_t*>(smem);         // whole batches of U steps, the last row repeated past the end
  for (int i = t; i < (steps + U - 1) / U * U * 16; i += 256) {
    const int j = min(j0 + i, j1 - 1);
    rows[i] = (uint32_t)(idx ? idx[j] : j) * (WIDE ? 1u : 2u * (uint32_t)Cout);
  }
  __syncthreads();
  const char* src = reinterpret_cast<const char*>(dY);
  const uint32_t colb = 2u * (uint32_t)min(c0 + 2 * x, Cout - 2);
  const bf16x2_t ones = __builtin_bit_cast(bf16x2_t, 0x3f803f80u);
  float s0 = 0.f, s1 = 0.f;
  auto batch = [&](int q0, auto last) {
    unsigned a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint2 r = *reinterpret_cast<const uint2*>(rows + 16 * (q0 + u) + 2 * y);
      const size_t ra = WIDE ? (size_t)r.x * (2u * (uint32_t)Cout) + colb : (size_t)(r.x + colb), rb = WIDE ? (size_t)r.y * (2u * (uint32_t)Cout) + colb : (size_t)(r.y + colb);
      a[u] = *reinterpret_cast<const unsigned*>(src + ra);
      b[u] = *reinterpret_cast<const unsigned*>(src + rb);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if constexpr (decltype(last)::value) {
        const int j = 16 * (q0 + u) + 2 * y;
        if (j >= n) a[u] = 0u;
        if (j + 1 >= n) b[u] = 0u;
      }
      s0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, (a[u] & 0xffffu) | (b[u] << 16)), ones, s0, false);
      s1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, (a[u] >> 16) | (b[u] & 0xffff0000u)), ones, s1, false);
    }
  };
  int q0 = 0;
  for (; 16 * (q0 + U) <= n; q0 += U) batch(q0, std::false_type{});
  if (q0 < steps) batch(q0, std::true_type{});
  __syncthreads();
  float(*red)[kColumns] = reinterpret_cast<float(*)[kColumns]>(smem);
  red[y][2 * x] = s0;
  red[y][2 * x + 1] = s1;
  __syncthreads();
  if (t < kColumns && c0 + t < Cout)
    dbp[c0 + t] = ((red[0][t] + red[1][t]) + (red[2][t] + red[3][t])) + ((red[4][t] + red[5][t]) + (red[6][t] + red[7][t]));
}

}  // namespace mid
}  // namespace sbp
#endif
