// Direct solve of the block-tridiagonal Schur system S lambda = gamma (14 states): the
// alternative to PCG for the Schur system of MPCGPU (Section III-B; the paper names a
// direct block-tridiagonal solve as future work, Section VI).  Exact up to rounding, FP64
// throughout, the same few launches whatever the conditioning:
//
//   direct_eliminate  a problem is cut into chunks of four knots, the first of them the
//       chunk's separator.  A wave forms its chunk's blocks from the inputs and eliminates
//       the three inner knots; what is left is a block-tridiagonal system of the separators.
//   sep_eliminate     the same elimination of the separators' system, four blocks to one,
//       while some problem has more than kCrBlocks of them.
//   separator_solve   block cyclic reduction of what is left, one workgroup per problem, in
//       LDS.
//   sep_back          a level's inner blocks from the next level's solution.
//   direct_back       lambda of the inner knots from the separators', then the primal step
//       dZ = -G^-1 (g - C^T lambda), or the adjoint gradients, one group per knot.
//
// Why this split: a block of S is 1.6 KB in FP64 against 1.4 KB of FP32 inputs for a whole
// knot, so a reduction that keeps S in memory is bound by re-reading it (a cyclic reduction
// over all knots moved ~13 blocks per knot).  Here S never leaves the compute unit, every Q,
// R and diagonal block is inverted once, and an inner knot writes only the two blocks its
// back substitution needs (W and H below).
//
// Elimination of inner knot k with D_k = S_kk after the previous step, T_k = A_k Q_k^-1
// (so S_{k+1,k} = -T_k) and F_k the coupling of k to the separator:
//   W_k = T_k D_k^-1,  H_k = F_k^T D_k^-1,  z_k = D_k^-1 y_k
//   D_{k+1} = S_{k+1,k+1} - W_k T_k^T,  y_{k+1} += T_k z_k,  F_{k+1}^T = H_k T_k^T
//   D_sep -= F_k^T H_k^T,  y_sep -= F_k^T z_k
//   lambda_k = z_k + W_k^T lambda_{k+1} - H_k^T lambda_sep
// The reduced matrices are Schur complements of S, so they stay positive definite; a pivot
// that is not > 0 means S is not (BREAKDOWN).
//
// Measured on MI355X against the formation kernel + cyclic reduction over all knots + primal
// step kernel it replaced: a forward and an adjoint of 256 problems of 17 to 500 knots (66,500
// in all) 1,587 -> 637 us, one problem of 128 knots 107 -> 47 us on the device, 256 of 128
// knots 372 -> 134 us.
#pragma once
#include "lane_ops.h"
#include "mpcpcg.h"
#include "pcg_kernel.h"

namespace mpc {

constexpr int kChunk = 4;  // knots per chunk (one per knot group of a wave)

// One chunk of a problem: of its knots (level 0) or of its separators (level 1, 2, ...).
struct Chunk {
  int64_t k0;    // first row of the problem at this level (packed knot, separator)
  int32_t N;     // knots, or separators, of the problem
  int32_t id;    // problem index b (x0 row, stats slot, control offset k0 - b)
  int32_t b0;    // first row of the chunk, its separator (a multiple of kChunk)
  int32_t sep;   // the separator among all
};

// The separators of one problem that separator_solve takes.
struct SepProb {
  int32_t sep0, nsep;
  int32_t id, N;
};

// The separators' systems, those of all levels numbered in one sequence: blocks by columns padded
// to kGroup rows (lane = row: a column is one line), vectors padded to kGroup.
struct SepRows {
  // the diagonal block: its own chunk's share, then the previous chunk's, [row][2][NX][kGroup];
  // -W^T and H^T in their place once the row is eliminated (a chunk's wave has moved both to
  // LDS by then, and nobody else reads them)
  double *d;
  double *l;        // the coupling to the previous separator
  double *yl, *yr;  // the right-hand side, two shares
  double *x;        // the solution
};

struct DirectArgs {
  // problem data (packed); q, r are the loss gradients dL/ddx, dL/ddu in the adjoint
  const float *Q, *R, *A, *B, *q, *r, *x0, *e, *gl;
  const float *lam_in, *dx_in, *du_in;
  float *lam, *dx, *du;
  float *dQ, *dR, *dA, *dB, *dq, *dr, *dx0, *de, *dgamma;
  mpcpcg_stats *stats;
  // schedule: the chunks of this launch's level, or (nullptr) those of one problem with N1
  // rows at that level, from row k0 to separators from sep0
  const Chunk *chunks;
  const SepProb *probs;
  int32_t nchunks, nprobs, N1;
  int32_t N;         // knots of the one problem
  int32_t k0, sep0;
  // what the elimination of this level's rows leaves: -W^T and H^T by columns
  // [rows][2][NX][kGroup] and z [rows][kGroup]
  double *wh, *z;
  SepRows sep;
  int32_t *flag;     // [problems] 1 once a pivot was not > 0 (0 between solves)
};

__device__ __forceinline__ Chunk chunk_of(const DirectArgs &a, int g) {
  if (a.chunks) return a.chunks[g];
  return Chunk{a.k0, a.N1, 0, g * kChunk, a.sep0 + g};
}
__device__ __forceinline__ SepProb sep_prob_of(const DirectArgs &a, int p) {
  if (a.probs) return a.probs[p];
  return SepProb{a.k0, a.N1, 0, a.N};
}

// ---------------------------------------------------------------- elimination
// One wave per chunk of four knots.  First each of the wave's four groups forms the blocks of
// its own knot (the same instructions for all four), then all four eliminate the inner knots
// one after the other together: every group solves with D_k for its four columns of each
// right-hand side.  With T'_k = S_{k+1,k} and the columns c of a group,
//   P_c = D_k^-1 (T'_k^T)_c,  R_c = D_k^-1 (F_k)_c          (-W_k^T and H_k^T)
//   (D_{k+1})_c -= T'_k P_c,  (F_{k+1})_c = -T'_k R_c,  (D_sep)_c -= F_k^T R_c
// a product's right operand is always the group's own columns, so only D_{k+1} and F_{k+1}
// pass through LDS, once per step.
// Bound by issue: ~3,400 vector instructions a chunk, 71% of the issue slots taken with three
// waves per SIMD (66,500 knots: 156 us, 335 MB).  A group per chunk instead needs a quarter
// fewer instructions, but four times the knots for the same waves: 27 instead of 14 us for
// one problem of 128 knots, and it measured no faster on the large batch (135 us, in rounds
// of 32,768 knots).
constexpr int kElimWaves = 4;  // chunks per workgroup (three workgroups per compute unit by LDS)
constexpr int kElimThreads = kElimWaves * 64;

// order this wave's LDS accesses: its earlier writes complete before its later reads
__device__ __forceinline__ void lds_order() {
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

template <int NX>
struct ElimShared {
  double T[kChunk - 1][NX][NX];  // T'_{k+1} = S_{k+2,k+1} by rows
  double D[kChunk][NX][NX];      // D_{k+1} by rows; the last is the next separator's share
  double F[NX][kGroup];          // F_k by columns
  double y[kChunk + 1][kGroup];
};

// Eliminates rows 1 .. 3 of the chunk whose blocks are in sh and whose separator's own
// diagonal block is in sep.d; writes the shares of the next level.
template <int NX>
__device__ __forceinline__ void eliminate_chunk(const DirectArgs &a, const Chunk &C, ElimShared<NX> &sh, int lane,
                                                int t, bool &pd) {
  const bool rowv = lane < NX;
  const int r = rowv ? lane : 0, N = C.N;
  constexpr int W = 4;                                   // columns per group
  int col[W];                                            // (clamped: the last group has two)
#pragma unroll
  for (int c = 0; c < W; ++c) col[c] = min(W * t + c, NX - 1);
  double Ds[W];                                          // the group's columns of D_sep
  double ys = sh.y[0][r];
#pragma unroll
  for (int c = 0; c < W; ++c) Ds[c] = a.sep.d[((int64_t)C.sep * 2 * NX + col[c]) * kGroup + lane];
#pragma unroll 1
  for (int k = 1; k < kChunk; ++k) {
    double D[NX], X[NX], P[2 * W + 1], O[2 * W];
#pragma unroll
    for (int j = 0; j < NX; ++j) D[j] = sh.D[k - 1][r][j];
#pragma unroll
    for (int c = 0; c < W; ++c) {
      P[c] = sh.T[k - 1][col[c]][r];
      P[W + c] = sh.F[col[c]][r];
    }
    P[2 * W] = sh.y[k][r];
    gj_solve<NX, 2 * W + 1>(D, P, lane, &pd);            // P_c, R_c and z
    const double z = P[2 * W];
#pragma unroll
    for (int j = 0; j < NX; ++j) X[j] = -sh.T[k - 1][r][j];
#pragma unroll
    for (int c = 0; c < W; ++c) {
      O[c] = sh.D[k][r][col[c]];
      O[W + c] = 0.0;
    }
    mm_nn_add<NX, 2 * W>(X, P, O);                       // D_{k+1} and F_{k+1}
    const double yn = sh.y[k + 1][r] + row_dot<NX>(X, z);
    // the sep's share: F_k^T rows are columns of F
    double Fr[NX];
#pragma unroll
    for (int j = 0; j < NX; ++j) Fr[j] = -sh.F[r][j];
    double R[W];
#pragma unroll
    for (int c = 0; c < W; ++c) R[c] = P[W + c];
    mm_nn_add<NX, W>(Fr, R, Ds);
    ys += row_dot<NX>(Fr, z);
    if (C.b0 + k < N) {
      double *wh = a.wh + ((C.k0 + C.b0 + k) * 2 * NX + W * t) * kGroup + lane;
#pragma unroll
      for (int c = 0; c < W; ++c)
        if (W * t + c < NX) {
          wh[c * kGroup] = P[c];
          wh[(NX + c) * kGroup] = P[W + c];
        }
      if (t == 0) a.z[(C.k0 + C.b0 + k) * kGroup + lane] = z;
    }
    lds_order();  // every read of D_{k+1} and F_k above is done
    if (rowv) {
#pragma unroll
      for (int c = 0; c < W; ++c)
        if (W * t + c < NX) {
          sh.D[k][lane][W * t + c] = O[c];
          sh.F[W * t + c][lane] = O[W + c];
        }
      sh.y[k + 1][lane] = yn;
    }
    lds_order();
  }
  // ---- the separator's own share, and the next separator's from this chunk
  const int64_t s = C.sep;
  const bool next = C.b0 + kChunk < N;
#pragma unroll
  for (int c = 0; c < W; ++c)
    if (W * t + c < NX) {
      const int64_t o = (s * 2 * NX + W * t + c) * kGroup + lane;
      a.sep.d[o] = Ds[c];
      if (next) {
        a.sep.d[o + 3 * NX * kGroup] = rowv ? sh.D[kChunk - 1][r][W * t + c] : 0.0;
        a.sep.l[((s + 1) * NX + W * t + c) * kGroup + lane] = rowv ? sh.F[W * t + c][r] : 0.0;
      }
    }
  if (t == 0) {
    a.sep.yl[s * kGroup + lane] = rowv ? ys : 0.0;
    if (next) a.sep.yr[(s + 1) * kGroup + lane] = rowv ? sh.y[kChunk][r] : 0.0;
  }
}

template <int NX, int NU, bool ADJ>
__global__ void __launch_bounds__(kElimThreads) direct_eliminate(const DirectArgs a) {
  static_assert(NX == 14, "four columns per group: 4 + 4 + 4 + 2");
  __shared__ __attribute__((aligned(16))) ElimShared<NX> shared[kElimWaves];
  const int lane = threadIdx.x & (kGroup - 1);
  const int t = (threadIdx.x >> 4) & 3;  // group: knot of the formation, column slice after it
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = blockIdx.x * kElimWaves + wave;
  if (g >= a.nchunks) return;  // whole waves leave; no workgroup barrier follows
  ElimShared<NX> &sh = shared[wave];
  const Chunk C = chunk_of(a, g);
  const int N = C.N, b = C.b0 + t;
  const bool rowv = lane < NX, act = b < N, ctl = b + 1 < N;
  const int64_t kb = C.k0 + b, cb = C.k0 - C.id + b;
  const int r = rowv ? lane : 0;
  bool pd = true;

  // ---- formation: Q_b^-1, T'_b = -A_b Q_b^-1 and theta's share of knot b + 1 (missing
  // blocks are zeros, missing Q and R identities)
  {
    double Qi[NX], Ab[NX], Bb[NU], Ri[NU];
#pragma unroll
    for (int j = 0; j < NX; ++j) { Qi[j] = (rowv && j == lane) ? 1.0 : 0.0; Ab[j] = 0.0; }
#pragma unroll
    for (int j = 0; j < NU; ++j) { Ri[j] = (j == lane) ? 1.0 : 0.0; Bb[j] = 0.0; }
    double qb = 0.0, rb = 0.0, add = 0.0;
    if (act && rowv) {
      const float *p = a.Q + (kb * NX + lane) * NX;
#pragma unroll
      for (int j = 0; j < NX; ++j) Qi[j] = (double)p[j];
      if (a.q) qb = (double)a.q[kb * NX + lane];
      if (ADJ)
        add = (double)a.gl[kb * NX + lane];
      else if (b == 0)
        add = (double)a.x0[(int64_t)C.id * NX + lane];
      else if (a.e)
        add = -(double)a.e[(cb - 1) * NX + lane];
    }
    if (ctl && rowv) {
      const float *p = a.A + (cb * NX + lane) * NX, *pb = a.B + (cb * NX + lane) * NU;
#pragma unroll
      for (int j = 0; j < NX; ++j) Ab[j] = (double)p[j];
#pragma unroll
      for (int j = 0; j < NU; ++j) Bb[j] = (double)pb[j];
    }
    if (ctl && lane < NU) {
      const float *p = a.R + (cb * NU + lane) * NU;
#pragma unroll
      for (int j = 0; j < NU; ++j) Ri[j] = (double)p[j];
      if (a.r) rb = (double)a.r[cb * NU + lane];
    }
    gj_inverse<NX>(Qi, lane);
    const double v = row_dot<NX>(Qi, qb);
    double yn = -row_dot<NX>(Ab, v);
    double T[NX], G[NX], U[NU];
    mm_nn<NX, NX>(Ab, Qi, T);
    mm_nt<NX, NX>(T, Ab, G);
    gj_inverse<NU>(Ri, lane);
    mm_nn<NU, NU>(Bb, Ri, U);
    mm_nt_add<NU, NX>(U, Bb, G);
    yn -= row_dot<NU>(U, rb);
    // D_{b+1} = Q_{b+1}^-1 + theta's share: this knot's G, then the next group's Q^-1 on top
    if (rowv) {
#pragma unroll
      for (int j = 0; j < NX; ++j) {
        if (t)
          sh.T[t - 1][lane][j] = -T[j];
        else
          sh.F[j][lane] = -T[j];  // F_1 = S_{1,0}
        sh.D[t][lane][j] = G[j];
      }
      sh.y[t + 1][lane] = yn;
    }
    if (t == 0)  // (a pad lane's row of Q^-1 is zero)
#pragma unroll
      for (int j = 0; j < NX; ++j) a.sep.d[((int64_t)C.sep * 2 * NX + j) * kGroup + lane] = Qi[j];
    lds_order();
    if (rowv) {
#pragma unroll
      for (int j = 0; j < NX; ++j)
        if (t) sh.D[t - 1][lane][j] += Qi[j];
      sh.y[t][lane] = t ? sh.y[t][lane] + (v + add) : v + add;
    }
    lds_order();
  }

  eliminate_chunk<NX>(a, C, sh, lane, t, pd);
  if (!pd) a.flag[C.id] = 1;  // every writer stores the same value
}

// The same for a chunk of four separators: S_{k+1,k} is the coupling L_{k+1}
// and the diagonal blocks are the sums of their two shares.
template <int NX>
__global__ void __launch_bounds__(kElimThreads) sep_eliminate(const DirectArgs a) {
  __shared__ __attribute__((aligned(16))) ElimShared<NX> shared[kElimWaves];
  const int lane = threadIdx.x & (kGroup - 1);
  const int t = (threadIdx.x >> 4) & 3;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = blockIdx.x * kElimWaves + wave;
  if (g >= a.nchunks) return;  // whole waves leave; no workgroup barrier follows
  ElimShared<NX> &sh = shared[wave];
  const Chunk C = chunk_of(a, g);
  const int b = C.b0 + t;
  const bool rowv = lane < NX, act = b < C.N, ctl = b + 1 < C.N;
  const int64_t k = C.k0 + (act ? b : C.b0), kn = ctl ? k + 1 : k;
  bool pd = true;
  {
    // rows past the horizon: identity diagonal, no coupling
    double D[NX], L[NX], G[NX];
    const double *pl = a.sep.l + kn * NX * kGroup + lane;
    const double *pd_ = a.sep.d + k * 2 * NX * kGroup + lane, *pr = pd_ + NX * kGroup;
    const bool two = act && b > 0;  // the first separator of a problem has one share
#pragma unroll
    for (int j = 0; j < NX; ++j) {
      D[j] = pd_[j * kGroup];
      G[j] = two ? pr[j * kGroup] : 0.0;
      L[j] = ctl ? pl[j * kGroup] : 0.0;
    }
    double y = act ? a.sep.yl[k * kGroup + lane] + (two ? a.sep.yr[k * kGroup + lane] : 0.0) : 0.0;
#pragma unroll
    for (int j = 0; j < NX; ++j) D[j] = act ? D[j] + G[j] : (j == lane ? 1.0 : 0.0);
    if (rowv) {
#pragma unroll
      for (int j = 0; j < NX; ++j) {
        if (t) {
          sh.T[t - 1][lane][j] = L[j];
          sh.D[t - 1][lane][j] = D[j];
        } else {
          sh.F[j][lane] = L[j];
          sh.D[kChunk - 1][lane][j] = 0.0;
        }
      }
      sh.y[t][lane] = y;
      if (t == 0) sh.y[kChunk][lane] = 0.0;
    }
    if (t == 0)
#pragma unroll
      for (int j = 0; j < NX; ++j) a.sep.d[((int64_t)C.sep * 2 * NX + j) * kGroup + lane] = rowv ? D[j] : 0.0;
    lds_order();
  }
  eliminate_chunk<NX>(a, C, sh, lane, t, pd);
  if (!pd) a.flag[C.id] = 1;
}

// ---------------------------------------------------------------- separators
// Block cyclic reduction.  With stride s (1, 2, 4, ...), the active blocks are the
// multiples of s; write L_i for the coupling of active block i to the active block before
// it and D_i for its diagonal block.  One level:
//   (a) every odd multiple j = s(2i+1) is eliminated:
//         V_j = D_j^-1 L_j,   U_j = D_j^-1 L_{j+s}^T,   z_j = D_j^-1 y_j;
//   (b) every even multiple i absorbs its eliminated neighbours j = i -+ s:
//         D_i -= L_i U_{i-s} + L_{i+s}^T V_{i+s},   y_i -= L_i z_{i-s} + L_{i+s}^T z_{i+s},
//         L_i <- -L_i V_{i-s}  (the coupling to i - 2s).
// When block 0 is the last one active, x_0 = D_0^-1 y_0, and the levels are undone in
// reverse order: x_j = z_j - V_j x_{j-s} - U_j x_{j+s}.
constexpr int kCrThreads = 512;
constexpr int kCrGroups = kCrThreads / kGroup, kCrWaves = kCrThreads / 64;

// dl holds D, then V once the block is eliminated (D_j is inverted in registers first); y
// turns into z.
//
// A whole wave works on one block task: its four groups split the columns of the products, a
// quarter of the chain.  Everything stays in LDS, where an exchange
// between sub-steps costs ~0.1 us instead of ~0.5 through memory.
constexpr int kCrBlocks = 32;  // separators of a problem that fit LDS
template <int NX>
struct CrShared {
  double dl[kCrBlocks][NX * NX], l[kCrBlocks][NX * NX], u[kCrBlocks][NX * NX];  // by columns
  double pad[kGroup];  // (lanes past the block's rows read up to two entries past its end)
  double y[kCrBlocks][kGroup], x[kCrBlocks][kGroup];
};

// Lanes past the block's rows (14, 15) hold copies of other rows or leftovers: nothing reads
// them across lanes, and they store nothing.
template <int NX>
struct CrOps {
  static constexpr int LD = NX;
  CrShared<NX> &st;
  const int n, lane, t;
  const bool rowv;
  __device__ __forceinline__ CrOps(CrShared<NX> &s_, int n_, int tid)
      : st(s_), n(n_), lane(tid & (kGroup - 1)), t((tid >> 4) & 3), rowv((tid & (kGroup - 1)) < NX) {}
  __device__ __forceinline__ void load(const double *blk, double (&o)[NX]) const {
#pragma unroll
    for (int c = 0; c < NX; ++c) o[c] = blk[c * LD + lane];
  }
  // row r of L^T, i.e. column r of L: contiguous per lane
  __device__ __forceinline__ const double *lt(int i) const { return st.l[i] + (rowv ? lane : 0) * LD; }
  __device__ __forceinline__ int n_odd(int s) const { return (n - s + 2 * s - 1) / (2 * s); }  // j = s(2i+1) < n
  __device__ __forceinline__ int n_even(int s) const { return (n - 1) / (2 * s) + 1; }         // i = 2sm < n

  // one wave: groups 0, 1 compute columns 0..6 and 7..13 of V_j, groups 2, 3 those of U_j
  __device__ __forceinline__ void odd(int j, int s, bool &pd) const {
    constexpr int H = NX / 2;
    double D[NX], C[H + 1];
    const int c0 = (t & 1) * H;
    const bool up = j + s < n;
    const bool isu = t >= 2 && up;
    const double *p = isu ? lt(j + s) + c0 : st.l[j] + c0 * LD + lane;
    const int step = isu ? 1 : LD;
    load(st.dl[j], D);
#pragma unroll
    for (int c = 0; c < H; ++c) C[c] = p[c * step];
    C[H] = st.y[j][lane];
    gj_solve<NX, H + 1>(D, C, lane, &pd);
    double *o = (t < 2 ? st.dl[j] : st.u[j]) + c0 * LD + lane;
    if (rowv && (t < 2 || up))
#pragma unroll
      for (int c = 0; c < H; ++c) o[c * LD] = C[c];
    if (t == 0 && rowv) st.y[j][lane] = C[H];
  }
  // one wave: L_i [U_{i-s} | V_{i-s}], seven columns a group; then L_{i+s}^T V_{i+s}, whose
  // inner sum of 14 terms is split between the wave's halves
  __device__ __forceinline__ void even(int i, int s) const {
    constexpr int H = NX / 2;
    const int c0 = (t & 1) * H, h = t >> 1;
    const bool left = i >= s, right = i + s < n;
    double D[H], A[H], B[H];
    const int col = c0 * LD + lane;
    double y = st.y[i][lane];
#pragma unroll
    for (int c = 0; c < H; ++c) {
      D[c] = st.dl[i][col + c * LD];
      A[c] = 0.0;
      B[c] = 0.0;
    }
    if (left) {
      double L[NX], T[H];
      load(st.l[i], L);
      const double *p = (h ? st.dl[i - s] : st.u[i - s]) + col;
#pragma unroll
      for (int c = 0; c < H; ++c) T[c] = p[c * LD];
      mm_nn_add<NX, H>(L, T, A);
      y -= row_dot<NX>(L, st.y[i - s][lane]);
    }
    if (right) {
      // rows 7h .. 7h + 6 of V_{i+s} on lanes 0 .. 6, and those entries of this lane's row of
      // L_{i+s}^T
      double X[H], T[H];
      const double *px = lt(i + s) + h * H;
      const int rv = min(lane + h * H, NX - 1);
      const double *p = st.dl[i + s] + c0 * LD + rv;
#pragma unroll
      for (int c = 0; c < H; ++c) {
        X[c] = px[c];
        T[c] = p[c * LD];
      }
      mm_nn_add<H, H>(X, T, B);
      const double part = row_dot<H>(X, st.y[i + s][rv]);
      y -= part + __shfl_xor(part, 32);
    }
#pragma unroll
    for (int c = 0; c < H; ++c) {
      const double o = __shfl_xor(B[c], 32);
      D[c] -= A[c] + (B[c] + o);
    }
    double *o = (h ? st.l[i] : st.dl[i]) + col;
    if (rowv && (!h || left))
#pragma unroll
      for (int c = 0; c < H; ++c) o[c * LD] = h ? -A[c] : D[c];
    if (t == 0 && rowv) st.y[i][lane] = y;
  }
  __device__ __forceinline__ void root(bool &pd) const {
    double D[NX], x[1] = {st.y[0][lane]};
    load(st.dl[0], D);
    gj_solve<NX, 1>(D, x, lane, &pd);
    if (t == 0 && rowv) st.x[0][lane] = x[0];
  }
  __device__ __forceinline__ void back(int j, int s) const {
    double T[NX];
    load(st.dl[j], T);
    double x = st.y[j][lane] - row_dot<NX>(T, st.x[j - s][lane]);
    if (j + s < n) {
      load(st.u[j], T);
      x -= row_dot<NX>(T, st.x[j + s][lane]);
    }
    if (rowv) st.x[j][lane] = x;
  }
  // one level, and one level of the back substitution, by the whole workgroup
  __device__ __forceinline__ void level(int s, bool &pd) const {
    const int wave = threadIdx.x / 64;
    const int no = n_odd(s), ne = n_even(s);
    for (int i = wave; i < no; i += kCrWaves) odd(s * (2 * i + 1), s, pd);
    __syncthreads();
    for (int i = wave; i < ne; i += kCrWaves) even(2 * s * i, s);
    __syncthreads();
  }
  __device__ __forceinline__ void level_back(int s) const {
    for (int i = threadIdx.x / kGroup; i < n_odd(s); i += kCrGroups) back(s * (2 * i + 1), s);
    __syncthreads();
  }
};

// One workgroup per problem; writes the problem's stats (direct_back turns a non-finite
// multiplier into BREAKDOWN as well) and clears its flag for the next solve.
template <int NX>
__global__ void __launch_bounds__(kCrThreads) separator_solve(const DirectArgs a) {
  __shared__ __attribute__((aligned(16))) CrShared<NX> sh;
  const SepProb P = sep_prob_of(a, blockIdx.x);
  const CrOps<NX> op(sh, P.nsep, threadIdx.x);
  bool pd = true;
  {  // one group per block, every load in flight at once
    static_assert(kCrThreads / kGroup >= kCrBlocks, "a group per block");
    const int lane = threadIdx.x & (kGroup - 1), i = threadIdx.x / kGroup;
    if (i < P.nsep && lane < NX) {
      const int64_t o = (int64_t)P.sep0 + i;
      double D[NX], R[NX], L[NX];
#pragma unroll
      for (int c = 0; c < NX; ++c) {
        D[c] = a.sep.d[(o * 2 * NX + c) * kGroup + lane];
        R[c] = i > 0 ? a.sep.d[((o * 2 + 1) * NX + c) * kGroup + lane] : 0.0;
        L[c] = i > 0 ? a.sep.l[(o * NX + c) * kGroup + lane] : 0.0;
      }
      sh.y[i][lane] = a.sep.yl[o * kGroup + lane] + (i > 0 ? a.sep.yr[o * kGroup + lane] : 0.0);
#pragma unroll
      for (int c = 0; c < NX; ++c) {
        sh.dl[i][c * NX + lane] = D[c] + R[c];
        sh.l[i][c * NX + lane] = L[c];
      }
    }
  }
  __syncthreads();
  int s = 1;
  for (; s < P.nsep; s *= 2) op.level(s, pd);
  if (threadIdx.x < 64) op.root(pd);
  __syncthreads();
  for (s /= 2; s >= 1; s /= 2) op.level_back(s);
  for (int i = threadIdx.x; i < P.nsep * kGroup; i += kCrThreads)
    a.sep.x[(int64_t)P.sep0 * kGroup + i] = i % kGroup < NX ? sh.x[i / kGroup][i % kGroup] : 0.0;
  const bool bad = __syncthreads_or(!pd) || a.flag[P.id] != 0;
  __syncthreads();  // every thread has read the flag
  if (threadIdx.x == 0) {
    a.flag[P.id] = 0;
    mpcpcg_stats st;
    st.iters = 0;
    st.status = bad ? MPCPCG_BREAKDOWN : MPCPCG_OK;
    st.final_ratio = 0.0f;
    st.reserved = 0;
    a.stats[P.id] = st;
  }
}

// ---------------------------------------------------------------- back substitution
// One wave per chunk, one group per row.  Every group loads its own W_i, H_i and z_i and
// forms z_i - H_i^T lambda_sep at once; only W_i^T lambda_{i+1} is a chain, which runs down
// the groups through LDS (14 fused multiply-adds a step).  Rows past the horizon get zeros.
constexpr int kBackThreads = 256;
constexpr int kBackWaves = kBackThreads / 64;

template <int NX>
__device__ __forceinline__ void chunk_back(const DirectArgs &a, const Chunk &C, double (&xs)[kChunk + 1][kGroup],
                                           int lane, int t) {
  const int N = C.N, b = C.b0 + t;
  const bool rowv = lane < NX;
  const int64_t s = C.sep;
  const double xl = a.sep.x[s * kGroup + lane];
  double W[NX], H[NX], u;
  if (t > 0 && b < N) {
    const double *w = a.wh + (C.k0 + b) * 2 * NX * kGroup + lane;  // rows of -W^T and H^T
#pragma unroll
    for (int j = 0; j < NX; ++j) {
      W[j] = w[j * kGroup];
      H[j] = w[(NX + j) * kGroup];
    }
    u = a.z[(C.k0 + b) * kGroup + lane];
  } else {
#pragma unroll
    for (int j = 0; j < NX; ++j) { W[j] = 0.0; H[j] = 0.0; }
    u = t == 0 ? xl : 0.0;
  }
  u -= row_dot<NX>(H, xl);
  if (t == 0) xs[kChunk][lane] = C.b0 + kChunk < N ? a.sep.x[(s + 1) * kGroup + lane] : 0.0;
  lds_order();
#pragma unroll
  for (int i = kChunk - 1; i >= 0; --i) {
    const double x = u - row_dot<NX>(W, xs[t + 1][lane]);
    if (t == i) xs[t][lane] = rowv ? x : 0.0;
    lds_order();
  }
}

// The inner blocks of a level of separators from the solution of the next level.
template <int NX>
__global__ void __launch_bounds__(kBackThreads) sep_back(const DirectArgs a) {
  __shared__ double shared[kBackWaves][kChunk + 1][kGroup];
  const int lane = threadIdx.x & (kGroup - 1), t = (threadIdx.x >> 4) & 3, wave = threadIdx.x >> 6;
  const int g = blockIdx.x * kBackWaves + wave;
  if (g >= a.nchunks) return;  // whole waves leave; no workgroup barrier follows
  const Chunk C = chunk_of(a, g);
  chunk_back<NX>(a, C, shared[wave], lane, t);
  if (C.b0 + t < C.N) a.sep.x[(C.k0 + C.b0 + t) * kGroup + lane] = shared[wave][t][lane];
}

// lambda of every knot, then the knot's primal step or gradients.
template <int NX, int NU, bool ADJ>
__global__ void __launch_bounds__(kBackThreads) direct_back(const DirectArgs a) {
  __shared__ double shared[kBackWaves][kChunk + 1][kGroup];
  const int lane = threadIdx.x & (kGroup - 1);
  const int t = (threadIdx.x >> 4) & 3;
  const int wave = threadIdx.x >> 6;
  const int g = blockIdx.x * kBackWaves + wave;
  if (g >= a.nchunks) return;  // whole waves leave; no workgroup barrier follows
  double (&xs)[kChunk + 1][kGroup] = shared[wave];
  const Chunk C = chunk_of(a, g);
  const int N = C.N, b = C.b0 + t;
  const bool rowv = lane < NX;
  chunk_back<NX>(a, C, xs, lane, t);
  const double lam = xs[t][lane], lamn = xs[t + 1][lane];
  const bool act = b < N, ctl = b + 1 < N;
  const int64_t kb = C.k0 + (act ? b : 0), cb = C.k0 - C.id + (ctl ? b : 0);
  // the knot's primal step: x_b = -Q_b^-1 (q_b - lambda_b + A_b^T lambda_{b+1}),
  // u_b = -R_b^-1 (r_b + B_b^T lambda_{b+1})
  double Qm[NX], Rm[NU];
  double xv = 0.0, uv = 0.0;
#pragma unroll
  for (int j = 0; j < NX; ++j) Qm[j] = (rowv && j == lane) ? 1.0 : 0.0;
#pragma unroll
  for (int j = 0; j < NU; ++j) Rm[j] = (j == lane) ? 1.0 : 0.0;
  if (act && rowv) {
    const float *p = a.Q + (kb * NX + lane) * NX;
#pragma unroll
    for (int j = 0; j < NX; ++j) Qm[j] = (double)p[j];
    xv = lam - (a.q ? (double)a.q[kb * NX + lane] : 0.0);
  }
  {
    double At[NX], Bt[NX];
#pragma unroll
    for (int j = 0; j < NX; ++j) { At[j] = 0.0; Bt[j] = 0.0; }
    if (ctl && rowv) {
      const float *p = a.A + cb * NX * NX + lane;
#pragma unroll
      for (int j = 0; j < NX; ++j) At[j] = (double)p[j * NX];
    }
    if (ctl && lane < NU) {
      const float *p = a.B + cb * NX * NU + lane;
#pragma unroll
      for (int j = 0; j < NX; ++j) Bt[j] = (double)p[j * NU];
      const float *pr = a.R + (cb * NU + lane) * NU;
#pragma unroll
      for (int j = 0; j < NU; ++j) Rm[j] = (double)pr[j];
      if (a.r) uv = -(double)a.r[cb * NU + lane];
    }
    xv -= row_dot<NX>(At, lamn);
    uv -= row_dot<NX>(Bt, lamn);
  }
  gj_solve<NX>(Qm, xv, lane);
  gj_solve<NU>(Rm, uv, lane);
  if (act && !(lam - lam == 0.0))  // infinite or not a number
    reinterpret_cast<int *>(a.stats + C.id)[1] = MPCPCG_BREAKDOWN;
  if constexpr (!ADJ) {
    if (act && rowv) {
      a.lam[kb * NX + lane] = (float)lam;
      a.dx[kb * NX + lane] = (float)xv;
    }
    if (ctl && lane < NU) a.du[cb * NU + lane] = (float)uv;
  } else {
    // lam holds mu, xv = nu1x_b, uv = nu1u_b
    double dxb = 0.0, ln = 0.0, dub = 0.0;
    if (act && rowv) dxb = (double)a.dx_in[kb * NX + lane];
    if (ctl && rowv) ln = (double)a.lam_in[(kb + 1) * NX + lane];
    if (ctl && lane < NU) dub = (double)a.du_in[cb * NU + lane];
    double P[NX], tmp[NX];
    // dQ_b = sym(nu1x_b dx_b^T); row i = (nu1x_i dx^T + dx_i nu1x^T) / 2
    outer_row<NX>(P, dxb, 0.5 * xv);
    outer_row<NX>(tmp, xv, 0.5 * dxb);
    if (act && rowv) {
      float *p = a.dQ + (kb * NX + lane) * NX;
#pragma unroll
      for (int j = 0; j < NX; ++j) p[j] = (float)(P[j] + tmp[j]);
      a.dq[kb * NX + lane] = (float)xv;
      if (a.dgamma) a.dgamma[kb * NX + lane] = (float)lam;
      if (b == 0) a.dx0[(int64_t)C.id * NX + lane] = (float)lam;
    }
    // dA_b = lambda_{b+1} nu1x_b^T + mu_{b+1} dx_b^T, dB_b likewise with the controls
    outer_row<NX>(P, xv, ln);
    outer_row<NX>(tmp, dxb, lamn);
    if (ctl && rowv) {
      float *p = a.dA + (cb * NX + lane) * NX;
#pragma unroll
      for (int j = 0; j < NX; ++j) p[j] = (float)(P[j] + tmp[j]);
      if (a.de) a.de[cb * NX + lane] = (float)(-lamn);
    }
    outer_row<NU>(P, uv, ln);
    outer_row<NU>(tmp, dub, lamn);
    if (ctl && rowv) {
      float *p = a.dB + (cb * NX + lane) * NU;
#pragma unroll
      for (int j = 0; j < NU; ++j) p[j] = (float)(P[j] + tmp[j]);
    }
    outer_row<NU>(P, dub, 0.5 * uv);
    outer_row<NU>(tmp, uv, 0.5 * dub);
    if (ctl && lane < NU) {
      float *p = a.dR + (cb * NU + lane) * NU;
#pragma unroll
      for (int j = 0; j < NU; ++j) p[j] = (float)(P[j] + tmp[j]);
      a.dr[cb * NU + lane] = (float)uv;
    }
  }
}

// The test hook of mpcpcg_debug_set_wait, launched only while it is set: these kernels wait for
// nothing across workgroups, so no time-out can be forced; a solved problem of more knots than
// one part of the PCG's (16) reports TIMEOUT all the same, any other keeps its status.
__global__ void __launch_bounds__(64) direct_stall_hook(const DirectArgs a) {
  const int p = blockIdx.x * 64 + threadIdx.x;
  if (p >= a.nprobs) return;
  const SepProb P = sep_prob_of(a, p);
  if (P.N > 16 && a.stats[P.id].status == MPCPCG_OK) a.stats[P.id].status = MPCPCG_TIMEOUT;
}

}  // namespace mpc
