// The 28-state / 14-control path.
//
// The 14-state kernel keeps each knot's rows of S and Phi^-1 in registers, one 16-lane
// DPP row per knot.  A 28-row block does not fit that mapping (a row of S is 84 FP64
// values), so this path stages the blocks in a device workspace instead.  Every kernel but
// the PCG gives a knot (a row of the block system) to a pair of 16-lane rows (pair_ops.h):
//   wide_form    Q^-1, S_{b+1,b}, the shares of S's diagonal blocks and right-hand sides;
//   for the PCG: wide_theta completes S_bb and forms D_b^-1; wide_precond forms Phi^-1 (FP32)
//                once every D^-1 exists; wide_pcg_gang (wide_pcg.h) is PCG (Algorithm 1) on
//                gangs of workgroups, rows of S and Phi^-1 in registers;
//   for the direct solve: wide_eliminate per level, wide_root, wide_back per level;
//   wide_epilogue  the primal step, or in adjoint mode nu_1 and the block-sparse gradients.
// Precision matches the 14-state kernel: FP64 formation, S, vectors and reductions; FP32
// Phi^-1.  Method references: S, gamma (Section III-B, sign-flipped so S is positive
// definite), Phi^-1 (Section IV-A), PCG (Algorithm 1), dZ = -G^-1 (g - C^T lambda).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mpcpcg.h"
#include "pair_ops.h"

namespace mpc {
namespace wide {

struct KnotDesc {    // one per knot of the packed batch
  int64_t k0;        // first knot row of the problem
  int32_t N;         // horizon of the problem
  int32_t b;         // knot index within the problem
  int32_t id;        // problem index
  int32_t pad;
};

struct WArgs {
  const float *Q, *R, *A, *B, *q, *r, *x0, *e;
  const float *lam_in, *dx_in, *du_in, *gl, *gx, *gu;
  float *lam, *dx, *du;
  mpcpcg_stats *stats;
  float *dQ, *dR, *dA, *dB, *dq, *dr, *dx0, *de, *dgamma;
  float *S_out, *P_out, *gam_out;
  const KnotDesc *knots;
  int32_t nknots;
  // workspace (FP64 unless noted; blocks by columns, so that the lanes that own a block's rows
  // move whole lines)
  double *S;      // [K][3][NX][NX]
  double *Dinv;   // [K][NX][NX]
  float *P;       // [K][3][NX][NX]
  double *rhs;    // [K][NX]; complete once wide_theta ran, before that without rhs_prev
  double *rhs_prev;  // [K][NX] the previous knot's share of the right-hand side
  double *Qinv;   // [K][NX][NX]
  float eps;
  int32_t max_iter;
  int32_t warm;
  int32_t adjoint;
  int32_t stop_abs;   // 1: eta < eps; 0: sqrt(eta / eta_ref) < eps
  int32_t need_up;    // 1: wide_form also writes S_{b,b+1} (the PCG reads it)
  int32_t direct;     // 1: wide_epilogue checks the multipliers (the PCG does it as it goes)
  double *lamw;       // [K][NX] lambda
};

// ---------------------------------------------------------------- formation
// wide_form: one pair of 16-lane rows per knot b (pair_ops.h; two knots per wave), each Q and
// R inverted once and nothing exchanged between knots:
//   Q_b^-1;  T = A_b Q_b^-1, written as S_{b+1,b} = -T and, transposed, as S_{b,b+1};
//   theta's share A_b Q_b^-1 A_b^T + B_b R_b^-1 B_b^T of knot b + 1 (to the place of S_{b+1,b+1});
//   gamma's (or the adjoint right-hand side's) share of b in rhs, of b + 1 in rhs_prev.
// wide_theta completes S_bb = share + Q_b^-1 and the right-hand side and forms D_b^-1 = S_bb^-1
// for the preconditioner; the direct solve adds the shares itself as it reads them.
// What bounds them is FP64 issue in one chain per wave and, before the blocks were laid out by
// columns, memory: a lane that walks its own row of 28 doubles touches one line per lane and
// entry.  Hence whole lines everywhere, and for the row-major inputs a detour through LDS.
// Measured on MI355X, 5,800 knots (a 32-problem two-arm batch), in us a direction:
//   wide_form   56, 66 with S_{b,b+1} for the PCG (one wave per knot, pivot rows by readlane,
//               products from LDS: 79, and 52 more for theta; one pair per knot with row-wise
//               access at 2 waves per SIMD: 105);
//   wide_theta  38 (with the products of theta and S before: 85); wide_precond 46 (130: one
//               workgroup per knot, operands in LDS);
//   wide_eliminate  110 for the knots, 43, 26 and 24 for the three levels above (odd-even
//               reduction, eight levels, blocks re-read on each: ~430); its blocks read when
//               needed and barriers that drained the stores: 164 for the knots, 55 a level;
//   wide_back 11 and 5 a level, wide_root 8;
//   wide_epilogue  37, after the PCG 45 (56 forward and 69 adjoint by one wave per knot).
// order this wave's LDS accesses: its earlier writes complete before its later reads
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

// a workgroup barrier for data in LDS: stores to global memory stay in flight across it
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

constexpr int kPairWaves = 2;  // waves per workgroup of the pair kernels

// indices of this thread's pair
struct PairLane {
  int lane, half, r, pr;  // lane of the 16-lane row, half, block row (clamped), pair of the wave
  bool rowv;
  __device__ __forceinline__ explicit PairLane(int tid)
      : lane(tid & 15), half((tid >> 4) & 1), r(14 * ((tid >> 4) & 1) + min(tid & 15, 13)), pr((tid >> 5) & 1),
        rowv((tid & 15) < 14) {}
};

// A block to the caller's row-major FP32 array: from the lanes' rows by way of a pair's LDS, whole
// lines (rows: this thread's row of the block; the pair's lanes all call it or none)
template <int NX>
__device__ __forceinline__ void put_block(float *out, float *lds, const double (&rows)[NX], const PairLane &L) {
  constexpr int MM = NX * NX;
  const int me = threadIdx.x & 31;
  wave_lds_order();
  if (L.rowv)
#pragma unroll
    for (int j = 0; j < NX; ++j) lds[L.r * NX + j] = (float)rows[j];
  wave_lds_order();
#pragma unroll 4
  for (int e = me; e < MM; e += 32) out[e] = lds[e];
}
template <int NX>
__device__ __forceinline__ void zero_block(float *out) {
  for (int e = threadIdx.x & 31; e < NX * NX; e += 32) out[e] = 0.0f;
}

// EXPORT (mpcpcg_form_schur): the three kernels of the preconditioner also write S, Phi^-1 and
// gamma of one problem as the caller's arrays.  Measured on MI355X, us a call in a row (alone, its
// inputs not in cache), 4, 64 and 512 knots: 42.0 (61.1), 42.2 (55.0), 45.5 (58.0); with a fourth
// launch that read them back from the workspace 44.1 (63.1), 48.2 (60.4), 60.0 (70.2); one wave
// per knot and a workgroup per knot for the preconditioner 52.0 (69.0), 54.0 (69.7), 70.0 (82.8).
template <int NX, int NU, bool EXPORT>
__global__ void __launch_bounds__(kPairWaves * 64) __attribute__((amdgpu_waves_per_eu(3, 3))) wide_form(const WArgs a) {
  static_assert(NX == pair::kN && NU == pair::kH, "blocks of 28 and 14 rows");
  constexpr int MM = NX * NX;
  const PairLane L(threadIdx.x);
  const int w = threadIdx.x >> 6;
  const int t = (blockIdx.x * kPairWaves + w) * 2 + L.pr;
  const bool live = t < a.nknots;
  const KnotDesc kd = a.knots[live ? t : a.nknots - 1];  // (a spare pair repeats the last knot)
  const int b = kd.b, r = L.r, lane = L.lane;
  const int64_t kb = kd.k0 + b;
  const int64_t cb = kd.k0 - kd.id + b;  // packed control row of control b
  const bool next = b + 1 < kd.N, out = live && L.rowv, outn = out && next;
  const bool adj = a.adjoint != 0;
  const float *qv = adj ? a.gx : a.q;
  const float *rv = adj ? a.gu : a.r;
  bool pd = true;
  double Qi[NX], v;
  // the input blocks arrive as they lie in memory, whole lines, and turn into rows through LDS
  constexpr int EM = (MM + 31) / 32, ER = (NU * NU + 31) / 32, EB = (NX * NU + 31) / 32;
  __shared__ __attribute__((aligned(16))) float stage[kPairWaves * 2][2][MM];
  float *s0 = stage[w * 2 + L.pr][0], *s1 = stage[w * 2 + L.pr][1];
  const int me = threadIdx.x & 31;
  float rv_[ER], bv_[EB];
  {
    float q[EM], f[EM];
#pragma unroll
    for (int j = 0; j < EM; ++j) {
      const int e = j * 32 + me;
      q[j] = e < MM ? a.Q[kb * MM + e] : 0.0f;
      f[j] = next && e < MM ? a.A[cb * MM + e] : 0.0f;
    }
#pragma unroll
    for (int j = 0; j < ER; ++j) rv_[j] = next && j * 32 + me < NU * NU ? a.R[cb * NU * NU + j * 32 + me] : 0.0f;
#pragma unroll
    for (int j = 0; j < EB; ++j) bv_[j] = next && j * 32 + me < NX * NU ? a.B[cb * NX * NU + j * 32 + me] : 0.0f;
#pragma unroll
    for (int j = 0; j < EM; ++j)
      if (j * 32 + me < MM) {
        s0[j * 32 + me] = q[j];
        s1[j * 32 + me] = f[j];
      }
  }
  wave_lds_order();
  {
    double Q[NX];
#pragma unroll
    for (int j = 0; j < NX; ++j) {
      Q[j] = (double)s0[r * NX + j];
      Qi[j] = j == r ? 1.0 : 0.0;
    }
    wave_lds_order();  // every row of Q has been read: R and B take its place
#pragma unroll
    for (int j = 0; j < ER; ++j)
      if (j * 32 + me < NU * NU) s0[j * 32 + me] = rv_[j];
#pragma unroll
    for (int j = 0; j < EB; ++j)
      if (j * 32 + me < NX * NU) s0[NU * NU + j * 32 + me] = bv_[j];
    pair::gj_solve<NX>(Q, Qi, lane, L.half, pd);
  }
  if (out)
#pragma unroll
    for (int j = 0; j < NX; ++j) a.Qinv[kb * MM + j * NX + r] = Qi[j];
  v = pair::row_dot(Qi, qv ? (double)qv[kb * NX + r] : 0.0);
  double add;
  if (adj) add = (double)a.gl[kb * NX + r];
  else if (b == 0) add = (double)a.x0[(int64_t)kd.id * NX + r];
  else add = a.e ? -(double)a.e[(cb - 1) * NX + r] : 0.0;
  if (out) {
    a.rhs[kb * NX + r] = v + add;
    double *S = a.S + kb * 3 * MM;
    if (b == 0) {  // no S_{0,-1} and no share of a previous knot
#pragma unroll
      for (int j = 0; j < NX; ++j) { S[j * NX + r] = 0.0; S[MM + j * NX + r] = 0.0; }
      a.rhs_prev[kb * NX + r] = 0.0;
    }
    if (!next)
#pragma unroll
      for (int j = 0; j < NX; ++j) S[2 * MM + j * NX + r] = 0.0;
  }
  if constexpr (EXPORT) {
    if (live && b == 0) zero_block<NX>(a.S_out + kb * 3 * MM);
    if (live && !next) zero_block<NX>(a.S_out + (kb * 3 + 2) * MM);
  }
  if (!__any(next)) return;
  double (&T)[NX] = Qi, G[NX], p1;  // T replaces Q^-1 column by column
  wave_lds_order();
  {
    double A[NX];
#pragma unroll
    for (int j = 0; j < NX; ++j) A[j] = (double)s1[r * NX + j];
    p1 = -pair::row_dot(A, v);
    pair::mm_inplace<NX>(A, T);
  }
#pragma unroll
  for (int j = 0; j < NX; ++j) G[j] = 0.0;
  pair::mm_nt_lds<NX>(T, s1, G);
  if (outn) {
    double *S0 = a.S + (kb + 1) * 3 * MM + r, *S2 = a.S + (kb * 3 + 2) * MM + r * NX;
#pragma unroll
    for (int j = 0; j < NX; ++j) {
      S0[j * NX] = -T[j];
      if (a.need_up) S2[j] = -T[j];
    }
  }
  if constexpr (EXPORT) {
    double V[NX];
#pragma unroll
    for (int j = 0; j < NX; ++j) V[j] = -T[j];
    if (live && next) put_block<NX>(a.S_out + (kb + 1) * 3 * MM, s1, V, L);  // (A_b has been used)
    if (outn)
#pragma unroll
      for (int j = 0; j < NX; ++j) a.S_out[(kb * 3 + 2) * MM + j * NX + r] = (float)V[j];
  }
  {
    // the control: both halves hold R^-1, each its rows of B
    double R[NU], B[NU], U[NU];
    const int ru = min(lane, NU - 1);
#pragma unroll
    for (int j = 0; j < NU; ++j) {
      R[j] = next ? (double)s0[ru * NU + j] : (j == ru ? 1.0 : 0.0);
      B[j] = (double)s0[NU * NU + r * NU + j];
    }
    gj_inverse<NU, 2>(R, lane, &pd);
    mm_nn<NU, NU>(B, R, U);
    pair::mm_nt_add<NU>(U, B, G);
    p1 -= mpc::row_dot<NU>(U, next && rv ? (double)rv[cb * NU + ru] : 0.0);
  }
  if (outn) {
    double *S1 = a.S + ((kb + 1) * 3 + 1) * MM + r;
#pragma unroll
    for (int j = 0; j < NX; ++j) S1[j * NX] = G[j];
    a.rhs_prev[(kb + 1) * NX + r] = p1;
  }
}

// S_bb, the right-hand side and D_b^-1 of knot b from the shares (D_0^-1 = S_00^-1 is Q_0
// itself).
template <int NX, bool EXPORT>
__global__ void __launch_bounds__(kPairWaves * 64) __attribute__((amdgpu_waves_per_eu(3, 3))) wide_theta(const WArgs a) {
  constexpr int MM = NX * NX;
  __shared__ float stage[EXPORT ? kPairWaves * 2 : 1][EXPORT ? MM : 1];
  const PairLane L(threadIdx.x);
  const int t = (blockIdx.x * kPairWaves + (threadIdx.x >> 6)) * 2 + L.pr;
  const bool live = t < a.nknots;
  const KnotDesc kd = a.knots[live ? t : a.nknots - 1];
  const int64_t kb = kd.k0 + kd.b;
  const int r = L.r;
  double *S1 = a.S + (kb * 3 + 1) * MM + r;
  double D[NX], I[NX];
  bool pd = true;
#pragma unroll
  for (int j = 0; j < NX; ++j) {
    D[j] = S1[j * NX] + a.Qinv[kb * MM + j * NX + r];
    I[j] = j == r ? 1.0 : 0.0;
  }
  const double y = a.rhs[kb * NX + r] + a.rhs_prev[kb * NX + r];
  if (live && L.rowv) {
    a.rhs[kb * NX + r] = y;
#pragma unroll
    for (int j = 0; j < NX; ++j) S1[j * NX] = D[j];
  }
  if constexpr (EXPORT)
    if (live) {
      put_block<NX>(a.S_out + (kb * 3 + 1) * MM, stage[threadIdx.x >> 5], D, L);
      if (L.rowv) a.gam_out[kb * NX + r] = (float)y;
    }
  if (__any(kd.b > 0)) pair::gj_solve<NX>(D, I, L.lane, L.half, pd);
  if (kd.b == 0)
#pragma unroll
    for (int j = 0; j < NX; ++j) I[j] = (double)a.Q[kb * MM + r * NX + j];
  if (live && L.rowv)
#pragma unroll
    for (int j = 0; j < NX; ++j) a.Dinv[kb * MM + j * NX + r] = I[j];
}

// Phi^-1 blocks, one pair per knot b (needs D^-1 of b and b + 1): D_b^-1 itself, and
// -D_{b+1}^-1 S_{b+1,b} D_b^-1, which is Phi^-1_{b+1,b} and, transposed, Phi^-1_{b,b+1}.  To the
// workspace by columns, or (EXPORT) only to the caller's array.
template <int NX, bool EXPORT>
__global__ void __launch_bounds__(kPairWaves * 64) __attribute__((amdgpu_waves_per_eu(3, 3))) wide_precond(const WArgs a) {
  constexpr int MM = NX * NX;
  __shared__ float stage[EXPORT ? kPairWaves * 2 : 1][EXPORT ? MM : 1];
  const PairLane L(threadIdx.x);
  const int t = (blockIdx.x * kPairWaves + (threadIdx.x >> 6)) * 2 + L.pr;
  const bool live = t < a.nknots;
  const KnotDesc kd = a.knots[live ? t : a.nknots - 1];
  const int64_t kb = kd.k0 + kd.b;
  const int r = L.r;
  const bool out = live && L.rowv, next = kd.b + 1 < kd.N;
  float *P = a.P + kb * 3 * MM + r;
  double D[NX], Y[NX];
#pragma unroll
  for (int j = 0; j < NX; ++j) D[j] = a.Dinv[kb * MM + j * NX + r];
  if constexpr (EXPORT) {
    if (live) {
      put_block<NX>(a.P_out + (kb * 3 + 1) * MM, stage[threadIdx.x >> 5], D, L);
      if (kd.b == 0) zero_block<NX>(a.P_out + kb * 3 * MM);
      if (!next) zero_block<NX>(a.P_out + (kb * 3 + 2) * MM);
    }
  } else if (out) {
#pragma unroll
    for (int j = 0; j < NX; ++j) {
      P[MM + j * NX] = (float)D[j];
      if (kd.b == 0) P[j * NX] = 0.0f;
      if (!next) P[2 * MM + j * NX] = 0.0f;
    }
  }
  if (!__any(next)) return;
  const int64_t kn = next ? kb + 1 : kb;
#pragma unroll
  for (int j = 0; j < NX; ++j) Y[j] = a.S[kn * 3 * MM + j * NX + r];  // S_{b+1,b}
  pair::mm_inplace<NX>(Y, D);
#pragma unroll
  for (int j = 0; j < NX; ++j) Y[j] = -a.Dinv[kn * MM + j * NX + r];
  pair::mm_inplace<NX>(Y, D);
  if constexpr (EXPORT) {
    if (live && next) put_block<NX>(a.P_out + kn * 3 * MM, stage[threadIdx.x >> 5], D, L);
    if (out && next)
#pragma unroll
      for (int j = 0; j < NX; ++j) a.P_out[(kb * 3 + 2) * MM + j * NX + r] = (float)D[j];
  } else if (out && next) {
    float *Pn = a.P + kn * 3 * MM + r, *Pu = a.P + (kb * 3 + 2) * MM + r * NX;
#pragma unroll
    for (int j = 0; j < NX; ++j) {
      Pn[j * NX] = (float)D[j];
      Pu[j] = (float)D[j];
    }
  }
}

// ---------------------------------------------------------------- direct solve
// The 14-state path's chunked elimination (tri_kernel.h has the recurrences) on 28-row blocks,
// four rows of a level to one until one is left per problem: level 0 are the knots, level
// l > 0 the separators of level l - 1.
//   wide_eliminate  one workgroup per chunk: it eliminates rows 1 .. 3 one after the other.  A
//       pair of 16-lane rows solves with D_k for W columns of T'_k^T or of F_k (and y_k), so
//       every pair repeats the elimination of D_k itself and the columns are spread over the
//       workgroup's 2 WAVES pairs.  Four waves (seven columns each, three workgroups per compute
//       unit): a level of few chunks is one chain of three eliminations, 25 us, and the knots'
//       level of the two-arm batch takes as long as with two waves and fourteen columns (less
//       repeated work, but a workgroup more to a compute unit): forward and adjoint 643 -> 626 us;
//   wide_root       the last separator of every problem, x_0 = D_0^-1 y_0, and its stats;
//   wide_back       the inner rows of a level from the next level's solution.
struct WChunk {
  int64_t k0;    // first row of the problem at this level
  int32_t N;     // rows of the problem
  int32_t id;    // problem
  int32_t b0;    // first row of the chunk, its separator
  int32_t sep;   // the separator's row at the next level
};

// The last row of a problem: a separator, or the problem's only knot.
struct WRoot {
  int64_t row;
  int32_t id;    // problem
  int32_t knot;  // 1: a knot
};

// The rows of one level: diagonal block (two shares), coupling to the previous row, right-hand
// side (two shares), solution; blocks by columns.  The separators of all levels above the knots
// are numbered in one sequence.
struct WLevel {
  double *d0, *d1, *l, *y0, *y1, *x;
  int64_t s0, s1, sl;  // doubles from one row's block to the next
  double *ph, *z;      // what this level's elimination leaves: -W^T | H^T by columns, z
  int64_t sp;          // doubles from one row's ph to the next
};

struct WDirect {
  const WChunk *chunks;
  WLevel in, out;
  int32_t *flag;
};

template <int NX, int WAVES>
__global__ void __launch_bounds__(WAVES * 64) __attribute__((amdgpu_waves_per_eu(3, 3))) wide_eliminate(const WDirect a) {
  constexpr int MM = NX * NX, W = NX / WAVES, LD = NX + 2;
  static_assert(NX == pair::kN && W % 7 == 0, "columns in blocks of seven");
  // by columns: D_1 .. D_3 (each takes the previous step's correction), and the couplings of
  // rows 1 .. 4 to their previous rows; the first of these becomes F_2, F_3
  __shared__ double Dk[3][NX][LD], Lk[4][NX][LD];
  double (&F)[NX][LD] = Lk[0];
  const PairLane L(threadIdx.x);
  const int slot = (threadIdx.x >> 6) * 2 + L.pr;
  const bool isF = slot >= WAVES;
  const int c0 = (isF ? slot - WAVES : slot) * W;
  const int lane = L.lane, half = L.half, r = L.r;
  const bool rowv = L.rowv;
  const WChunk C = a.chunks[blockIdx.x];
  const int N = C.N;
  bool pd = true;
  double Ds[W], yk[4], yc = 0.0;  // the F slots' columns of the separator's diagonal block; y_0 .. y_3
  {
    const int64_t k0 = C.k0 + C.b0;
    constexpr int per = (MM / 2 + WAVES * 64 - 1) / (WAVES * 64);
    double2 d0[3][per], d1[3][per], l[4][per];
    const int left = N - C.b0;
#pragma unroll
    for (int q = 0; q < per; ++q) {
      const int e = q * WAVES * 64 + threadIdx.x;
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const bool on = e < MM / 2 && m + 1 < left;
        if (m < 3) {
          d0[m][q] = on ? reinterpret_cast<const double2 *>(a.in.d0 + (k0 + 1 + m) * a.in.s0)[e] : double2{0.0, 0.0};
          d1[m][q] = on ? reinterpret_cast<const double2 *>(a.in.d1 + (k0 + 1 + m) * a.in.s1)[e] : double2{0.0, 0.0};
        }
        l[m][q] = on ? reinterpret_cast<const double2 *>(a.in.l + (k0 + 1 + m) * a.in.sl)[e] : double2{0.0, 0.0};
      }
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) yk[m] = m < left ? a.in.y0[(k0 + m) * NX + r] + a.in.y1[(k0 + m) * NX + r] : 0.0;
#pragma unroll
    for (int c = 0; c < W; ++c)
      Ds[c] = a.in.d0[k0 * a.in.s0 + r + (c0 + c) * NX] + a.in.d1[k0 * a.in.s1 + r + (c0 + c) * NX];
#pragma unroll
    for (int q = 0; q < per; ++q) {
      const int e = q * WAVES * 64 + threadIdx.x, at = e / (NX / 2) * LD + e % (NX / 2) * 2;
      if (e < MM / 2)
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          if (m < 3)
            *reinterpret_cast<double2 *>(&Dk[m][0][0] + at) = double2{d0[m][q].x + d1[m][q].x, d0[m][q].y + d1[m][q].y};
          *reinterpret_cast<double2 *>(&Lk[m][0][0] + at) = l[m][q];
        }
    }
  }
  double ys = yk[0], O[W];
  lds_barrier();
#pragma unroll 1
  for (int k = 1; k < 4; ++k) {
    const int i = C.b0 + k;
    if (i >= N) break;  // (the same for the whole workgroup)
    double b[W + 1];
    {
      double D[NX];
#pragma unroll
      for (int j = 0; j < NX; ++j) D[j] = Dk[k - 1][j][r];
#pragma unroll
      for (int c = 0; c < W; ++c) b[c] = isF ? F[c0 + c][r] : Lk[k][r][c0 + c];
      b[W] = yk[1] + yc;
      yk[1] = yk[2];
      yk[2] = yk[3];
      pair::gj_solve<W + 1>(D, b, lane, half, pd);       // -W^T or H^T columns, and z
    }
    const double z = b[W];
    if (rowv) {
      // (in the place of row i's own shares of the diagonal block, which the whole workgroup
      // had moved to LDS before its first barrier and nobody else reads)
      double *o = a.in.ph + (C.k0 + i) * a.in.sp + (isF ? MM : 0) + c0 * NX + r;
#pragma unroll
      for (int c = 0; c < W; ++c) o[c * NX] = b[c];
      if (slot == 0) a.in.z[(C.k0 + i) * NX + r] = z;
    }
    double X[NX];
#pragma unroll
    for (int j = 0; j < NX; ++j) X[j] = -F[r][j];        // -(F_k^T)
    if (isF) pair::mm_add<W>(X, b, Ds);
    ys += pair::row_dot(X, z);
#pragma unroll
    for (int j = 0; j < NX; ++j) X[j] = -Lk[k][j][r];
#pragma unroll
    for (int c = 0; c < W; ++c) O[c] = 0.0;
    pair::mm_add<W>(X, b, O);                            // D_{k+1}'s correction, or F_{k+1}
    yc = pair::row_dot(X, z);
    if (k == 3) break;
    lds_barrier();
    if (rowv)
#pragma unroll
      for (int c = 0; c < W; ++c) {
        if (isF)
          F[c0 + c][r] = O[c];
        else
          Dk[k][c0 + c][r] += O[c];
      }
    lds_barrier();
  }
  const int64_t s = C.sep;
  if (rowv) {
    if (isF)
#pragma unroll
      for (int c = 0; c < W; ++c) a.out.d0[s * a.out.s0 + (c0 + c) * NX + r] = Ds[c];
    if (slot == 0) a.out.y0[s * NX + r] = ys;
    if (C.b0 == 0) {  // a problem's first separator has no share from a previous chunk
      if (!isF)
#pragma unroll
        for (int c = 0; c < W; ++c) a.out.d1[s * a.out.s1 + (c0 + c) * NX + r] = 0.0;
      if (slot == 0) a.out.y1[s * NX + r] = 0.0;
    }
    if (C.b0 + 4 < N) {
#pragma unroll
      for (int c = 0; c < W; ++c) {
        if (isF)
          a.out.l[(s + 1) * a.out.sl + (c0 + c) * NX + r] = O[c];
        else
          a.out.d1[(s + 1) * a.out.s1 + (c0 + c) * NX + r] = O[c];
      }
      if (slot == 0) a.out.y1[(s + 1) * NX + r] = yc;
    }
  }
  if (!pd) a.flag[C.id] = 1;  // every writer stores the same value
}

// The last row of each problem: x = D^-1 y, the stats, and the breakdown flag cleared for the next
// solve (wide_epilogue turns a non-finite multiplier into BREAKDOWN as well).
template <int NX>
__global__ void __launch_bounds__(64) wide_root(const WArgs a, const WLevel knots, const WLevel seps, const WRoot *roots,
                                                int nprobs, int32_t *flag) {
  const PairLane L(threadIdx.x);
  const int p = blockIdx.x * 2 + L.pr;
  const bool live = p < nprobs;
  const WRoot P = roots[live ? p : nprobs - 1];
  const int64_t k = P.row;
  const WLevel v = P.knot ? knots : seps;
  double D[NX], y[1];
  bool pd = true;
#pragma unroll
  for (int j = 0; j < NX; ++j) D[j] = v.d0[k * v.s0 + L.r + j * NX] + v.d1[k * v.s1 + L.r + j * NX];
  y[0] = v.y0[k * NX + L.r] + v.y1[k * NX + L.r];
  pair::gj_solve<1>(D, y, L.lane, L.half, pd);
  if (live && L.rowv) v.x[k * NX + L.r] = y[0];
  const unsigned long long bad = __ballot(!pd) >> (32 * L.pr) & 0xffffffffull;
  if (live && (threadIdx.x & 31) == 0) {
    mpcpcg_stats st;
    st.iters = 0;
    st.status = bad || flag[P.id] ? MPCPCG_BREAKDOWN : MPCPCG_OK;
    st.final_ratio = 0.0f;
    st.reserved = 0;
    a.stats[P.id] = st;
    flag[P.id] = 0;
  }
}

// One workgroup per chunk, one pair per row: z - H^T x_sep at once, then the chain
// x_i = z_i - H_i^T x_sep + W_i^T x_{i+1} down the rows through LDS.
template <int NX>
__global__ void __launch_bounds__(128) wide_back(const WDirect a) {
  constexpr int MM = NX * NX;
  __shared__ double xs[5][32];
  const PairLane L(threadIdx.x);
  const int t = (threadIdx.x >> 6) * 2 + L.pr, r = L.r, me = threadIdx.x & 31;
  const WChunk C = a.chunks[blockIdx.x];
  const int i = C.b0 + t;
  const int64_t s = C.sep;
  const double xl = a.out.x[s * NX + r];
  double P[NX], u = t == 0 ? xl : 0.0;
  const bool inner = t > 0 && i < C.N;
  const double *ph = a.in.ph + (C.k0 + (inner ? i : C.b0)) * a.in.sp + r;
#pragma unroll
  for (int j = 0; j < NX; ++j) P[j] = inner ? ph[MM + j * NX] : 0.0;
  if (inner) u = a.in.z[(C.k0 + i) * NX + r];
  u -= pair::row_dot(P, xl);
#pragma unroll
  for (int j = 0; j < NX; ++j) P[j] = inner ? ph[j * NX] : 0.0;
  if (t == 0) xs[4][me] = C.b0 + 4 < C.N ? a.out.x[(s + 1) * NX + r] : 0.0;
  __syncthreads();
#pragma unroll
  for (int q = 3; q >= 0; --q) {
    const double x = u - pair::row_dot(P, xs[t + 1][me]);
    if (t == q) xs[t][me] = x;
    __syncthreads();
  }
  if (i < C.N && L.rowv) a.in.x[(C.k0 + i) * NX + r] = xs[t][me];
}

// ---------------------------------------------------------------- primal step, gradients
// One pair per knot b, from the multipliers lamw (lambda, or mu in adjoint mode):
//   x_b = Q_b^-1 (lambda_b - q_b - A_b^T lambda_{b+1}),  u_b = -R_b^-1 (r_b + B_b^T lambda_{b+1})
// and in adjoint mode, with (x, u) = nu_1, the block-sparse gradients.  Matrices are read and
// written by columns of row-major arrays: lane r takes column r, consecutive addresses.
template <int NX, int NU>
__global__ void __launch_bounds__(kPairWaves * 64) wide_epilogue(const WArgs a) {
  constexpr int MM = NX * NX;
  const PairLane L(threadIdx.x);
  const int t = (blockIdx.x * kPairWaves + (threadIdx.x >> 6)) * 2 + L.pr;
  const bool live = t < a.nknots;
  const KnotDesc kd = a.knots[live ? t : a.nknots - 1];
  const int b = kd.b, r = L.r, lane = L.lane;
  const int64_t kb = kd.k0 + b;
  const int64_t cb = kd.k0 - kd.id + b;  // control b
  const bool next = b + 1 < kd.N, out = live && L.rowv, outn = out && next;
  const bool adj = a.adjoint != 0;
  const float *qv = adj ? a.gx : a.q;
  const float *rv = adj ? a.gu : a.r;
  const double lam = a.lamw[kb * NX + r], ln = next ? a.lamw[(kb + 1) * NX + r] : 0.0;
  if (a.direct && out && !(lam - lam == 0.0))  // infinite or not a number
    reinterpret_cast<int *>(a.stats + kd.id)[1] = MPCPCG_BREAKDOWN;
  double x, u;
  {
    double M[NX];
#pragma unroll
    for (int j = 0; j < NX; ++j) M[j] = next ? (double)a.A[cb * MM + j * NX + r] : 0.0;
    const double w = lam - (qv ? (double)qv[kb * NX + r] : 0.0) - pair::row_dot(M, ln);
#pragma unroll
    for (int j = 0; j < NX; ++j) M[j] = a.Qinv[kb * MM + j * NX + r];
    x = pair::row_dot(M, w);
  }
  const int c = min(lane, NU - 1);  // control row / column of this lane, the same in both halves
  {
    double M[NX], R[NU];
#pragma unroll
    for (int j = 0; j < NX; ++j) M[j] = next ? (double)a.B[cb * NX * NU + j * NU + c] : 0.0;
#pragma unroll
    for (int j = 0; j < NU; ++j) R[j] = next ? (double)a.R[cb * NU * NU + c * NU + j] : (j == c ? 1.0 : 0.0);
    u = -((next && rv ? (double)rv[cb * NU + c] : 0.0) + pair::row_dot(M, ln));
    gj_solve<NU, 2>(R, u, lane);
  }
  const bool outu = live && next && lane < NU && L.half == 0;
  if (!adj) {
    if (out) {
      a.lam[kb * NX + r] = (float)lam;
      a.dx[kb * NX + r] = (float)x;
    }
    if (outu) a.du[cb * NU + lane] = (float)u;
    return;
  }
  if (out) {
    if (a.dgamma) a.dgamma[kb * NX + r] = (float)lam;
    a.dq[kb * NX + r] = (float)x;
    if (b == 0) a.dx0[(int64_t)kd.id * NX + r] = (float)lam;
  }
  if (outu) a.dr[cb * NU + lane] = (float)u;
  if (outn && a.de) a.de[cb * NX + r] = (float)(-ln);
  const double dx = (double)a.dx_in[kb * NX + r];
  // rows 14 h .. 14 h + 13 of column r, the row vector's halves on every lane of the pair
  auto half_rows = [&](double s0, double v0, double s1, double v1, double (&C)[NU], int h) {
    double lo, hi;
#pragma unroll
    for (int k = 0; k < NU; ++k) C[k] = 0.0;
    pair::dup(s0, lo, hi);
    outer_row_add<NU>(C, h ? hi : lo, v0);
    pair::dup(s1, lo, hi);
    outer_row_add<NU>(C, h ? hi : lo, v1);
  };
  double C[NU];
  // dQ_b = sym(nu1x_b dx_b^T)
  for (int h = 0; h < 2; ++h) {
    half_rows(dx, 0.5 * x, x, 0.5 * dx, C, h);
    if (out)
#pragma unroll
      for (int k = 0; k < NU; ++k) a.dQ[kb * MM + (14 * h + k) * NX + r] = (float)C[k];
  }
  if (!__any(next)) return;
  // dA_b = lambda_{b+1} nu1x_b^T + mu_{b+1} dx_b^T, dB_b = lambda_{b+1} nu1u_b^T + mu_{b+1} du_b^T,
  // dR_b = sym(nu1u_b du_b^T)
  const double li = next ? (double)a.lam_in[(kb + 1) * NX + r] : 0.0;
  const double du = next ? (double)a.du_in[cb * NU + c] : 0.0;
  for (int h = 0; h < 2; ++h) {
    half_rows(li, x, ln, dx, C, h);
    if (outn)
#pragma unroll
      for (int k = 0; k < NU; ++k) a.dA[cb * MM + (14 * h + k) * NX + r] = (float)C[k];
  }
  half_rows(li, u, ln, du, C, 0);
  {
    double C1[NU];
    half_rows(li, u, ln, du, C1, 1);  // each half writes its rows of B's columns
    if (live && next && lane < NU)
#pragma unroll
      for (int k = 0; k < NU; ++k) a.dB[cb * NX * NU + (14 * L.half + k) * NU + lane] = (float)(L.half ? C1[k] : C[k]);
  }
#pragma unroll
  for (int k = 0; k < NU; ++k) C[k] = 0.0;
  outer_row_add<NU>(C, du, 0.5 * u);
  outer_row_add<NU>(C, u, 0.5 * du);
  if (outu)
#pragma unroll
    for (int k = 0; k < NU; ++k) a.dR[cb * NU * NU + k * NU + lane] = (float)C[k];
}

}  // namespace wide
}  // namespace mpc
