// Lane-level building blocks for 16-lane "knot groups" on CDNA4 (gfx950).
//
// A knot group is one 16-lane DPP row of a wave64.  Lane i of the group owns row i of
// every nx x nx block of its knot (rows >= nx hold zeros), so a matrix is NX registers
// per lane and a vector is one register per lane.  Products broadcast a row of the
// right-hand operand from its owner lane with DPP row_newbcast, which never leaves the
// 16-lane row, so four knots per wave run without interfering.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "dpp_asm.h"

namespace mpc {

constexpr int kGroup = 16;          // lanes per knot group (one DPP row)
constexpr int kRowNewBcast = 0x150; // DPP row_newbcast:n  (broadcast lane n of each row)
constexpr int kRowShr = 0x110;      // DPP row_shr:n       (lane i <- lane i-n, zero fill)

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xF, 0xF, true);
  const uint32_t hi =
      (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// value of v in lane K of this lane's 16-lane group
template <int K>
__device__ __forceinline__ double bc(double v) { return dpp_f64<kRowNewBcast + K>(v); }
template <int K>
__device__ __forceinline__ float bcf(float v) { return dpp_f32<kRowNewBcast + K>(v); }

// Sum over the 16 lanes of the group; the full sum lands in lane 15 (other lanes hold
// partial prefix sums).
__device__ __forceinline__ double group_sum_to_last(double v) {
  v += dpp_f64<kRowShr + 1>(v);
  v += dpp_f64<kRowShr + 2>(v);
  v += dpp_f64<kRowShr + 4>(v);
  v += dpp_f64<kRowShr + 8>(v);
  return v;
}

// group_sum_to_last of two values, their steps interleaved (each rounds as on its own).
__device__ __forceinline__ void group_sums2(double &a, double &b) {
  a += dpp_f64<kRowShr + 1>(a);
  b += dpp_f64<kRowShr + 1>(b);
  a += dpp_f64<kRowShr + 2>(a);
  b += dpp_f64<kRowShr + 2>(b);
  a += dpp_f64<kRowShr + 4>(a);
  b += dpp_f64<kRowShr + 4>(b);
  a += dpp_f64<kRowShr + 8>(a);
  b += dpp_f64<kRowShr + 8>(b);
}

// 64-bit DPP move with a row mask: lanes of rows outside ROWS get 0.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_f64_rows(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWS, 0xF, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROWS, 0xF, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
constexpr int kRowBcast15 = 0x142;  // DPP row_bcast:15 (lane 15 of a row to the next row)

// Two 32-lane sums at once: lanes 0..31 carry the terms of the first sum, lanes 32..63
// those of the second.  Each is g0 + g1 of its two 16-lane row sums (fixed shape); both
// results are uniform (read from lanes 31 and 63).  One reduction chain serves both sums.
__device__ __forceinline__ void half_sums(double v, double &s0, double &s1) {
  double g = group_sum_to_last(v);
  g += dpp_f64_rows<kRowBcast15, 0xA>(g);  // rows 1, 3: + lane 15 of rows 0, 2
  const uint64_t u = __builtin_bit_cast(uint64_t, g);
  const uint32_t lo0 = __builtin_amdgcn_readlane((uint32_t)u, 31);
  const uint32_t hi0 = __builtin_amdgcn_readlane((uint32_t)(u >> 32), 31);
  const uint32_t lo1 = __builtin_amdgcn_readlane((uint32_t)u, 63);
  const uint32_t hi1 = __builtin_amdgcn_readlane((uint32_t)(u >> 32), 63);
  s0 = __builtin_bit_cast(double, ((uint64_t)hi0 << 32) | lo0);
  s1 = __builtin_bit_cast(double, ((uint64_t)hi1 << 32) | lo1);
}

// Sum over the 64 lanes of the wave with a fixed reduction shape (identical rounding in
// every wave that calls it); the result is returned in every lane.
__device__ __forceinline__ double wave_sum(double v) {
  const double g = group_sum_to_last(v);
  const uint64_t u = __builtin_bit_cast(uint64_t, g);
  const uint32_t lo = (uint32_t)u, hi = (uint32_t)(u >> 32);
  double s = 0.0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t l2 = __builtin_amdgcn_readlane(lo, 16 * q + 15);
    const uint32_t h2 = __builtin_amdgcn_readlane(hi, 16 * q + 15);
    s += __builtin_bit_cast(double, ((uint64_t)h2 << 32) | l2);
  }
  return s;
}

// ---- hot-loop matvec rows with the broadcast fused into the FMA -----------------------
// acc += sum_{j<NX} m[j] * x(lane j).  One asm block per 14-term row keeps the DPP
// broadcast folded into v_fmac (the compiler does not fuse row_newbcast by itself).  The
// leading s_nop covers the VALU-write -> DPP-read hazard on x, which the compiler cannot
// see through inline asm; x is not written inside the block.
// Operand %0 is the accumulator, %1 the broadcast source and %2..%15 the matrix
// entries; term K multiplies matrix operand K+2 by x broadcast from lane K.
#define MPC_F64_T(K, OP) "v_fmac_f64_dpp %0, %1, %" #OP " row_newbcast:" #K " row_mask:0xf bank_mask:0xf\n"
#define MPC_F32_T(K, OP) "v_fmac_f32_dpp %0, %1, %" #OP " row_newbcast:" #K " row_mask:0xf bank_mask:0xf\n"

__device__ __forceinline__ void row_fma14_f64(double &acc, double x, const double (&m)[14]) {
  asm volatile("s_nop 1\n" MPC_F64_T(0, 2) MPC_F64_T(1, 3) MPC_F64_T(2, 4) MPC_F64_T(3, 5)
                   MPC_F64_T(4, 6) MPC_F64_T(5, 7) MPC_F64_T(6, 8) MPC_F64_T(7, 9)
                       MPC_F64_T(8, 10) MPC_F64_T(9, 11) MPC_F64_T(10, 12) MPC_F64_T(11, 13)
                           MPC_F64_T(12, 14) MPC_F64_T(13, 15)
               : "+&v"(acc)
               : "v"(x), "v"(m[0]), "v"(m[1]), "v"(m[2]), "v"(m[3]), "v"(m[4]), "v"(m[5]),
                 "v"(m[6]), "v"(m[7]), "v"(m[8]), "v"(m[9]), "v"(m[10]), "v"(m[11]),
                 "v"(m[12]), "v"(m[13]));
}

__device__ __forceinline__ void row_fma14_f32(float &acc, float x, const float (&m)[14]) {
  asm volatile("s_nop 1\n" MPC_F32_T(0, 2) MPC_F32_T(1, 3) MPC_F32_T(2, 4) MPC_F32_T(3, 5)
                   MPC_F32_T(4, 6) MPC_F32_T(5, 7) MPC_F32_T(6, 8) MPC_F32_T(7, 9)
                       MPC_F32_T(8, 10) MPC_F32_T(9, 11) MPC_F32_T(10, 12) MPC_F32_T(11, 13)
                           MPC_F32_T(12, 14) MPC_F32_T(13, 15)
               : "+&v"(acc)
               : "v"(x), "v"(m[0]), "v"(m[1]), "v"(m[2]), "v"(m[3]), "v"(m[4]), "v"(m[5]),
                 "v"(m[6]), "v"(m[7]), "v"(m[8]), "v"(m[9]), "v"(m[10]), "v"(m[11]),
                 "v"(m[12]), "v"(m[13]));
}

// ---- small dense algebra on row-distributed matrices ---------------------------------
// All products go through the fused blocks of dpp_asm.h.  Sizes are 14 (state) or
// 7 (control) for the Kuka-shaped problems this library is built for.

template <int n> struct DAsm;
template <> struct DAsm<14> {
  template <int LM> static __device__ __forceinline__ void rowdot(double &acc, double x, const double (&M)[LM]) { dasm::rowdot14(acc, x, M); }
  template <int LC> static __device__ __forceinline__ void outer(double (&C)[LC], double s, double x) { dasm::outer14(C, s, x); }
};
template <> struct DAsm<7> {
  template <int LM> static __device__ __forceinline__ void rowdot(double &acc, double x, const double (&M)[LM]) { dasm::rowdot7(acc, x, M); }
  template <int LC> static __device__ __forceinline__ void outer(double (&C)[LC], double s, double x) { dasm::outer7(C, s, x); }
};

// sum_{k<K} m[k] * x(lane k)  (row of a matrix times a lane-distributed vector)
template <int K, int L>
__device__ __forceinline__ double row_dot(const double (&m)[L], double x) {
  double acc = 0.0;
  DAsm<K>::rowdot(acc, x, m);
  return acc;
}

// C += X Y on J columns (Y's rows owned by lanes m), one block: a single pair of wait states
// instead of one per row of Y
template <int M, int J, int LX, int LY, int LC>
__device__ __forceinline__ void mm_nn_add(const double (&X)[LX], const double (&Y)[LY],
                                          double (&C)[LC]) {
  if constexpr (M == 14 && J == 14) dasm::prod14x14(C, Y, X);
  else if constexpr (M == 14 && J == 8) dasm::prod14x8(C, Y, X);
  else if constexpr (M == 14 && J == 7) dasm::prod14x7(C, Y, X);
  else if constexpr (M == 14 && J == 4) dasm::prod14x4(C, Y, X);
  else {
    static_assert(M == 7 && J == 7, "no block of this shape");
    dasm::prod7x7(C, Y, X);
  }
}

// C = X Y : C[j] = sum_{m<M} X[m] Y(lane m)[j], j < J   (Y's rows owned by lanes m)
template <int M, int J, int LX, int LY, int LC>
__device__ __forceinline__ void mm_nn(const double (&X)[LX], const double (&Y)[LY],
                                      double (&C)[LC]) {
#pragma unroll
  for (int j = 0; j < J; ++j) C[j] = 0.0;
  mm_nn_add<M, J>(X, Y, C);
}

// C += X Y^T : C[j] += sum_{m<M} X[m] Y(lane j)[m], j < J   (Y's rows owned by lanes j)
template <int M, int J, int LX, int LY, int LC>
__device__ __forceinline__ void mm_nt_add(const double (&X)[LX], const double (&Y)[LY],
                                          double (&C)[LC]) {
  static_assert(J == 14 && (M == 14 || M == 7), "no block of this shape");
  if constexpr (M == 14) dasm::prodt14x14(C, Y, X);
  else dasm::prodt7x14(C, Y, X);
}
// C = X Y^T
template <int M, int J, int LX, int LY, int LC>
__device__ __forceinline__ void mm_nt(const double (&X)[LX], const double (&Y)[LY],
                                      double (&C)[LC]) {
#pragma unroll
  for (int j = 0; j < J; ++j) C[j] = 0.0;
  mm_nt_add<M, J>(X, Y, C);
}

// C[k] += s(lane k) * x for k < n
template <int n, int LC>
__device__ __forceinline__ void outer_row_add(double (&C)[LC], double s, double x) {
  DAsm<n>::outer(C, s, x);
}
// C[k] = s(lane k) * x for k < n  (a broadcast vector scaled by a lane value)
template <int n, int LC>
__device__ __forceinline__ void outer_row(double (&C)[LC], double s, double x) {
#pragma unroll
  for (int k = 0; k < n; ++k) C[k] = 0.0;
  DAsm<n>::outer(C, s, x);
}

// One elimination step a_j += bc_k(a_j) * c over CNT columns of a: the columns col(0), ...,
// col(CNT - 1) of a compile-time map, in one block.
template <int k, int CNT, class COL>
__device__ __forceinline__ void elim_cols(COL &&col, double c) {
  static_assert(CNT >= 0 && CNT <= 7, "columns per block");
  using std::integral_constant;
  auto at = [&](auto r) -> double & { return col(r); };
#define MPC_C(R) at(integral_constant<int, R>{})
  if constexpr (CNT == 1) dasm::elim<k>(MPC_C(0), c);
  if constexpr (CNT == 2) dasm::elim<k>(MPC_C(0), MPC_C(1), c);
  if constexpr (CNT == 3) dasm::elim<k>(MPC_C(0), MPC_C(1), MPC_C(2), c);
  if constexpr (CNT == 4) dasm::elim<k>(MPC_C(0), MPC_C(1), MPC_C(2), MPC_C(3), c);
  if constexpr (CNT == 5) dasm::elim<k>(MPC_C(0), MPC_C(1), MPC_C(2), MPC_C(3), MPC_C(4), c);
  if constexpr (CNT == 6) dasm::elim<k>(MPC_C(0), MPC_C(1), MPC_C(2), MPC_C(3), MPC_C(4), MPC_C(5), c);
  if constexpr (CNT == 7) dasm::elim<k>(MPC_C(0), MPC_C(1), MPC_C(2), MPC_C(3), MPC_C(4), MPC_C(5), MPC_C(6), c);
#undef MPC_C
}
// columns AT .. AT + CNT - 1
template <int k, int AT, int CNT, int L>
__device__ __forceinline__ void elim_tail(double (&a)[L], double c) {
  elim_cols<k, CNT>([&](auto r) -> double & { return a[AT + decltype(r)::value]; }, c);
}
// entries AT .. AT + CNT - 1 of the columns 0 .. n-1 without k and k + 1
template <int n, int k, int AT, int CNT, int L>
__device__ __forceinline__ void elim_rest(double (&a)[L], double c) {
  elim_cols<k, CNT>(
      [&](auto r) -> double & {
        constexpr int i = AT + decltype(r)::value;
        return a[k + 1 < n && i >= k ? i + 2 : i];
      },
      c);
}

// Reciprocal: hardware estimate + Newton steps, without the division's scaling and fix-up
// sequence.  Measured on MI355X over 2^20 values (largest relative error): the estimate 2^-24.4,
// one step 2^-48.7 (on average 2^-52.9), two steps 2^-53, the same doubles as a division.
__device__ __forceinline__ double newton_f64(double x, double d) {
  return __builtin_fma(d, __builtin_fma(-x, d, 1.0), d);
}
template <int STEPS = 1>
__device__ __forceinline__ double rcp_f64(double x) {
  double d = __builtin_amdgcn_rcp(x);
#pragma unroll
  for (int i = 0; i < STEPS; ++i) d = newton_f64(x, d);
  return d;
}

// In-place Gauss-Jordan inverse of an n x n symmetric positive definite matrix whose row
// `lane` is a[0..n-1] (rows >= n must be zero and stay zero).  No pivoting is needed for
// SPD matrices: every pivot is a positive Schur complement.  Step k: every row i but the
// pivot row loses f_i = a_ik / a_kk times the pivot row, and column k becomes 1 in the
// pivot row and -f_i elsewhere; the pivot row itself is left unscaled and every row is
// multiplied by its own 1 / a_ii once at the end, so a step costs one fused multiply-add
// per column.  A chain of 14 dependent pivots bounds it: column k + 1 is updated first, and
// the next pivot's reciprocal (STEPS Newton steps) runs beside the updates of the other columns.
// `positive` (optional) ends false on a lane whose row's pivot is not > 0: the matrix is
// positive definite if it stays true on every lane.
template <int n, int STEPS = 1, int L>
__device__ __forceinline__ void gj_inverse(double (&a)[L], int lane, bool *positive = nullptr) {
  static_assert(STEPS == 1 || STEPS == 2, "one or two Newton steps");
  double piv = bc<0>(a[0]);
  double d = rcp_f64<STEPS>(piv);
  double mine = 0.0;  // 1 / a_ii of this lane's row
  static_for<0, n>([&](auto kk) {
    constexpr int k = decltype(kk)::value;
    const bool me = (lane == k);
    const double f = a[k] * d;
    const double c = me ? 0.0 : -f;
    mine = me ? d : mine;
    a[k] = me ? 1.0 : c;
    constexpr int rest = k + 1 < n ? n - 2 : n - 1;
    if constexpr (k + 1 < n) {
      dasm::elim<k>(a[k + 1], c);
      piv = bc<k + 1>(a[k + 1]);
      d = __builtin_amdgcn_rcp(piv);
      elim_rest<n, k, 0, rest / 2>(a, c);
      d = newton_f64(piv, d);
      elim_rest<n, k, rest / 2, rest - rest / 2>(a, c);
      if constexpr (STEPS == 2) d = newton_f64(piv, d);
    } else {
      elim_rest<n, k, 0, rest / 2>(a, c);
      elim_rest<n, k, rest / 2, rest - rest / 2>(a, c);
    }
  });
  if (positive) *positive = *positive && (lane >= n || mine > 0.0);
#pragma unroll
  for (int j = 0; j < n; ++j) a[j] *= mine;
}

// b <- a^-1 b for an n x n symmetric positive definite matrix whose row `lane` is a (rows
// >= n zero, a is consumed) and m right-hand sides whose row `lane` is b: the elimination
// above on the columns right of each pivot and on b only.  For m columns of a product a^-1 b
// it costs n (n / 2 + m) multiply-adds a lane instead of the inverse's n^2 and the product's
// n m.
template <int n, int m, int STEPS = 1, int L>
__device__ __forceinline__ void gj_solve(double (&a)[L], double (&b)[m], int lane, bool *positive = nullptr) {
  static_assert(STEPS == 1 || STEPS == 2, "one or two Newton steps");
  double piv = bc<0>(a[0]);
  double d = rcp_f64<STEPS>(piv);
  double mine = 0.0;
  static_for<0, n>([&](auto kk) {
    constexpr int k = decltype(kk)::value;
    const bool me = (lane == k);
    const double c = me ? 0.0 : -(a[k] * d);
    mine = me ? d : mine;
    constexpr int left = n - 2 - k;  // columns k + 2 .. n - 1
    if constexpr (k + 1 < n) {
      dasm::elim<k>(a[k + 1], c);
      piv = bc<k + 1>(a[k + 1]);
      d = __builtin_amdgcn_rcp(piv);
    }
    elim_tail<k, 0, (m > 7 ? 7 : m)>(b, c);
    if constexpr (m > 7) elim_tail<k, 7, m - 7>(b, c);
    if constexpr (k + 1 < n) d = newton_f64(piv, d);
    if constexpr (left > 0) {
      elim_tail<k, k + 2, (left + 1) / 2>(a, c);
      elim_tail<k, k + 2 + (left + 1) / 2, left / 2>(a, c);
    }
    if constexpr (k + 1 < n && STEPS == 2) d = newton_f64(piv, d);
  });
  if (positive) *positive = *positive && (lane >= n || mine > 0.0);
#pragma unroll
  for (int j = 0; j < m; ++j) b[j] *= mine;
}
template <int n, int STEPS = 1, int L>
__device__ __forceinline__ void gj_solve(double (&a)[L], double &x, int lane) {
  double b[1] = {x};
  gj_solve<n, 1, STEPS>(a, b, lane);
  x = b[0];
}

}  // namespace mpc
