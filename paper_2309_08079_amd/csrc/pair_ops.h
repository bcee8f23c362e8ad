// Lane-level building blocks for 28-row blocks on CDNA4 (gfx950).
//
// A "pair" is two neighbouring 16-lane DPP rows: lane i < 14 of the first row owns row i of a
// 28 x 28 block, lane i < 14 of the second row owns row 14 + i (the first and second half of
// the block), all 28 entries of a row in one lane's registers.  DPP row_newbcast reaches only
// the lanes of its own 16-lane row, so the rows of a right-hand operand are first copied to
// both halves with v_permlane16_swap (one move and one swap per 32-bit register give both
// copies), and products then run as the 14-row blocks of dpp_asm.h do.  A wave holds two
// pairs.  Lanes 14 and 15 of a row hold nothing that other lanes read.
#pragma once
#include "lane_ops.h"

namespace mpc {
namespace pair {

// (the blocks are large: without this the compiler leaves the lambdas as calls and their
// arrays in scratch)
#define MPC_INLINE __attribute__((always_inline))

constexpr int kN = 28;  // rows of a block
constexpr int kH = 14;  // rows of a half

// v of the first half and of the second half, on the lanes of both
__device__ __forceinline__ void dup(double v, double &lo, double &hi) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t a = (uint32_t)u, b = (uint32_t)(u >> 32);
  const auto x = __builtin_amdgcn_permlane16_swap(a, a, false, false);
  const auto y = __builtin_amdgcn_permlane16_swap(b, b, false, false);
  lo = __builtin_bit_cast(double, ((uint64_t)y[0] << 32) | x[0]);
  hi = __builtin_bit_cast(double, ((uint64_t)y[1] << 32) | x[1]);
}

// (M x)_r, x distributed over the lanes
__device__ __forceinline__ double row_dot(const double (&M)[kN], double x) {
  double lo, hi, m0[kH], m1[kH];
  dup(x, lo, hi);
#pragma unroll
  for (int j = 0; j < kH; ++j) { m0[j] = M[j]; m1[j] = M[kH + j]; }
  return mpc::row_dot<kH>(m0, lo) + mpc::row_dot<kH>(m1, hi);
}

// C[j] += sum_m X[m] Y(row m)[j] for j < J, J a multiple of 7
template <int J, int LY, int LC>
__device__ __forceinline__ void mm_add(const double (&X)[kN], const double (&Y)[LY], double (&C)[LC]) {
  static_assert(J % 7 == 0 && J <= LY && J <= LC, "columns in blocks of seven");
  double x0[kH], x1[kH];
#pragma unroll
  for (int j = 0; j < kH; ++j) { x0[j] = X[j]; x1[j] = X[kH + j]; }
  static_for<0, J / 7>([&](auto q) MPC_INLINE {
    constexpr int c = 7 * decltype(q)::value;
    double lo[7], hi[7], acc[7];
#pragma unroll
    for (int j = 0; j < 7; ++j) {
      dup(Y[c + j], lo[j], hi[j]);
      acc[j] = C[c + j];
    }
    mm_nn_add<kH, 7>(x0, lo, acc);
    mm_nn_add<kH, 7>(x1, hi, acc);
#pragma unroll
    for (int j = 0; j < 7; ++j) C[c + j] = acc[j];
  });
}

// Y <- X Y, in place
template <int J, int LY>
__device__ __forceinline__ void mm_inplace(const double (&X)[kN], double (&Y)[LY]) {
  static_assert(J % 7 == 0 && J <= LY, "columns in blocks of seven");
  double x0[kH], x1[kH];
#pragma unroll
  for (int j = 0; j < kH; ++j) { x0[j] = X[j]; x1[j] = X[kH + j]; }
  static_for<0, J / 7>([&](auto q) MPC_INLINE {
    constexpr int c = 7 * decltype(q)::value;
    double lo[7], hi[7], acc[7];
#pragma unroll
    for (int j = 0; j < 7; ++j) {
      dup(Y[c + j], lo[j], hi[j]);
      acc[j] = 0.0;
    }
    mm_nn_add<kH, 7>(x0, lo, acc);
    mm_nn_add<kH, 7>(x1, hi, acc);
#pragma unroll
    for (int j = 0; j < 7; ++j) Y[c + j] = acc[j];
  });
}

// C[j] += sum_m X[m] Y[j][m] for all 28 rows j, Y row-major FP32 in LDS
template <int M>
__device__ __forceinline__ void mm_nt_lds(const double (&X)[kN], const float *Y, double (&C)[kN]) {
  static_assert(M % 7 == 0 && M <= kN, "terms in blocks of seven");
  const int i = min((int)(threadIdx.x & 15), kH - 1) * kN;
  double c0[kH], c1[kH];
#pragma unroll
  for (int j = 0; j < kH; ++j) { c0[j] = C[j]; c1[j] = C[kH + j]; }
  static_for<0, M / 7>([&](auto q) MPC_INLINE {
    constexpr int m = 7 * decltype(q)::value;
    double lo[7], hi[7], x[7];
#pragma unroll
    for (int j = 0; j < 7; ++j) {
      lo[j] = (double)Y[i + m + j];
      hi[j] = (double)Y[kH * kN + i + m + j];
      x[j] = X[m + j];
    }
    dasm::prodt7x14(c0, lo, x);
    dasm::prodt7x14(c1, hi, x);
  });
#pragma unroll
  for (int j = 0; j < kH; ++j) { C[j] = c0[j]; C[kH + j] = c1[j]; }
}

// C[j] += sum_{m < M} X[m] Y(row j)[m] for all 28 rows j (X times Y^T), M a multiple of 7
template <int M, int LX, int LY>
__device__ __forceinline__ void mm_nt_add(const double (&X)[LX], const double (&Y)[LY], double (&C)[kN]) {
  static_assert(M % 7 == 0 && M <= LX && M <= LY, "terms in blocks of seven");
  double c0[kH], c1[kH];
#pragma unroll
  for (int j = 0; j < kH; ++j) { c0[j] = C[j]; c1[j] = C[kH + j]; }
  static_for<0, M / 7>([&](auto q) MPC_INLINE {
    constexpr int m = 7 * decltype(q)::value;
    double lo[7], hi[7], x[7];
#pragma unroll
    for (int j = 0; j < 7; ++j) {
      dup(Y[m + j], lo[j], hi[j]);
      x[j] = X[m + j];
    }
    dasm::prodt7x14(c0, lo, x);
    dasm::prodt7x14(c1, hi, x);
  });
#pragma unroll
  for (int j = 0; j < kH; ++j) { C[j] = c0[j]; C[kH + j] = c1[j]; }
}

// columns AT .. END - 1 of an elimination step
template <int k, int AT, int END, int L>
__device__ __forceinline__ void elim_range(double (&a)[L], double c) {
  if constexpr (AT < END) {
    constexpr int n = END - AT > 7 ? 7 : END - AT;
    elim_tail<k, AT, n>(a, c);
    elim_range<k, AT + n, END>(a, c);
  }
}

// Gauss-Jordan elimination of the 14 pivots of half H from the rows of that half: columns
// FROM.. of a and all of b; the other half's rows are left as they are.  The pivots'
// reciprocals are rounded as a division's (two Newton steps): 28 pivots a block and up to three
// blocks a chunk and level follow one another, and one step costs up to five bits of each.
template <int H, int W>
__device__ __forceinline__ void eliminate_half(double (&a)[kN], double (&b)[W], int lane, int half, bool &pd) {
  constexpr int O = H * kH;
  const bool on = half == H;
  double piv = bc<0>(a[O]);
  double d = rcp_f64<2>(piv);
  double mine = 1.0;
  static_for<0, kH>([&](auto kk) MPC_INLINE {
    constexpr int k = decltype(kk)::value;
    const bool me = lane == k;
    const double c = me || !on ? 0.0 : -(a[O + k] * d);
    mine = me && on ? d : mine;
    constexpr int first = O + k + 1;  // columns first .. 27
    if constexpr (k + 1 < kH) {
      dasm::elim<k>(a[first], c);
      piv = bc<k + 1>(a[first]);
      d = __builtin_amdgcn_rcp(piv);
    }
    elim_range<k, 0, W>(b, c);
    if constexpr (k + 1 < kH) d = newton_f64(piv, d);
    elim_range<k, (k + 1 < kH ? first + 1 : first), kN>(a, c);
    if constexpr (k + 1 < kH) d = newton_f64(piv, d);
  });
  pd = pd && (!on || lane >= kH || mine > 0.0);
  if constexpr (H == 0)
#pragma unroll
    for (int j = kH; j < kN; ++j) a[j] *= mine;
#pragma unroll
  for (int j = 0; j < W; ++j) b[j] *= mine;
}

// b <- a^-1 b for a symmetric positive definite 28 x 28 matrix (a is consumed) and W right-hand
// sides: with a = [P Q; Q^T R] the first half solves Z = P^-1 [Q | b], the second half takes
// R - Q^T Z and solves it, and the first half's rows get the second's solution.  Half of the
// lanes work at a time, but a pivot row never leaves its DPP row.
template <int W>
__device__ __forceinline__ void gj_solve(double (&a)[kN], double (&b)[W], int lane, int half, bool &pd) {
  eliminate_half<0, W>(a, b, lane, half, pd);
  double x[kH];
  auto columns = [&](auto &v, auto at, auto cnt, auto use_hi) MPC_INLINE {
    constexpr int A = decltype(at)::value, C = decltype(cnt)::value;
    double y[7], acc[7];
#pragma unroll
    for (int j = 0; j < 7; ++j) {
      double lo = 0.0, hi = 0.0;
      if (j < C) dup(v[A + (j < C ? j : 0)], lo, hi);
      y[j] = decltype(use_hi)::value ? hi : lo;
      acc[j] = j < C ? v[A + (j < C ? j : 0)] : 0.0;
    }
    if constexpr (C == 7)
      mm_nn_add<kH, 7>(x, y, acc);
    else if constexpr (C == 1)
      acc[0] += mpc::row_dot<kH>(x, y[0]);
    else
      static_assert(C == 7 || C == 1, "right-hand sides in blocks of seven and one");
#pragma unroll
    for (int j = 0; j < C; ++j) v[A + j] = acc[j];
  };
  using std::integral_constant;
#pragma unroll
  for (int j = 0; j < kH; ++j) x[j] = half ? -a[j] : 0.0;
  static_for<0, 2>([&](auto q) MPC_INLINE { columns(a, integral_constant<int, kH + 7 * decltype(q)::value>{}, integral_constant<int, 7>{}, integral_constant<bool, false>{}); });
  static_for<0, W / 7>([&](auto q) MPC_INLINE { columns(b, integral_constant<int, 7 * decltype(q)::value>{}, integral_constant<int, 7>{}, integral_constant<bool, false>{}); });
  static_for<W / 7 * 7, W>([&](auto q) MPC_INLINE { columns(b, q, integral_constant<int, 1>{}, integral_constant<bool, false>{}); });
  eliminate_half<1, W>(a, b, lane, half, pd);
#pragma unroll
  for (int j = 0; j < kH; ++j) x[j] = half ? 0.0 : -a[kH + j];
  static_for<0, W / 7>([&](auto q) MPC_INLINE { columns(b, integral_constant<int, 7 * decltype(q)::value>{}, integral_constant<int, 7>{}, integral_constant<bool, true>{}); });
  static_for<W / 7 * 7, W>([&](auto q) MPC_INLINE { columns(b, q, integral_constant<int, 1>{}, integral_constant<bool, true>{}); });
}

}  // namespace pair
}  // namespace mpc
