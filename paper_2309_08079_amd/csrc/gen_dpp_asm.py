"""Writes dpp_asm.h: the fused DPP-broadcast FMA blocks of the knot-group kernels.

Each block is one inline-asm statement of v_fmac_f64_dpp instructions with a row_newbcast
source, for rows of 14 (states) and 7 (controls) or slices of them.  The shapes differ only
in operand numbering and the broadcast lane, so they are generated here rather than
written by hand.  Run `python gen_dpp_asm.py` in this folder after
editing; tests/test_abi_cpu.py checks that the committed header is this script's output.
"""
from __future__ import annotations

import os
import sys

HEADER = """\
// Fused DPP-broadcast FMA blocks (v_fmac_f64_dpp with row_newbcast).
// Generated by gen_dpp_asm.py in this folder: edit the generator, not this file.
//
// Accumulators are early-clobber ("+&v"): a block writes them before it has read every
// input, so they must not share a register with any input.
// Every block starts with "s_nop 1": the hardware needs two wait states between a VALU
// write of a VGPR and a DPP read of it, and the compiler cannot see DPP reads inside
// inline asm.  No DPP source is written inside a block.  Keeping the broadcast inside the
// FMA also stops the compiler from hoisting hundreds of broadcast copies (and spilling).
//
// Shapes (lane i of a 16-lane group; bc_k(v) = v in lane k of the group):
//   rowdot(acc, x, M): acc += sum_k bc_k(x) * M[k]      k < n   (row of M dot vector x)
//   outer(C, s, x):    C[k] += bc_k(s) * x              k < n   (vector s scaled by x)
//   prodMxN(C, Y, X):  C[j] += sum_k bc_k(Y[j]) * X[k]   j < N, k < M   (X times Y, N columns)
//   prodtMxN(C, Y, X): C[j] += sum_k bc_j(Y[k]) * X[k]   j < N, k < M   (X times Y^T)
//   elim<K>(a0, ..., c): a_j += bc_K(a_j) * c, 1 to 7 columns in place (an elimination
//                      step: a lane's DPP source is read in the instruction that writes
//                      it, and no column is read twice inside a block)
#pragma once

namespace mpc {
namespace dasm {
"""

FOOTER = """
}  // namespace dasm
}  // namespace mpc
"""

LANES = 14  # broadcast lanes a block may name (rows of the largest block)


def insn(t, dst, src0, src1, lane):
    """One fused FMA: dst += bc_lane(src0) * src1 (operand numbers)."""
    return '"v_fmac_%s_dpp %%%d, %%%d, %%%d row_newbcast:%d row_mask:0xf bank_mask:0xf\\n"' % (
        t, dst, src0, src1, lane)


def asm(insns, outs, ins, tail=""):
    return 'asm volatile("s_nop 1\\n" %s%s : %s : %s);' % ("".join(insns), tail, ", ".join(outs), ", ".join(ins))


def per_lane(name, targs, sig, assertion, body_of_k):
    lines = ["template <%s>" % targs, "__device__ __forceinline__ void %s(%s) {" % (name, sig),
             "  static_assert(%s, \"shape\");" % assertion]
    for k in range(LANES):
        head = "if constexpr (K == %d)" % k if k == 0 else "else if constexpr (K == %d)" % k
        lines.append("  %s { %s }" % (head, body_of_k(k)))
    lines.append("}")
    return lines


def vectors(T, t, n):
    """Products of a row with a lane-distributed vector, and the outer product's row."""
    C = ['"+&v"(C[%d])' % j for j in range(n)]
    M = ['"v"(M[%d])' % j for j in range(n)]
    return ["template <int LM>",
            "__device__ __forceinline__ void rowdot%d(%s &acc, %s x, const %s (&M)[LM]) {" % (n, T, T, T),
            "  static_assert(LM >= %d, \"shape\");" % n,
            "  " + asm([insn(t, 0, 1, 2 + k, k) for k in range(n)], ['"+&v"(acc)'], ['"v"(x)'] + M),
            "}",
            "template <int LC>",
            "__device__ __forceinline__ void outer%d(%s (&C)[LC], %s s, %s x) {" % (n, T, T, T),
            "  static_assert(LC >= %d, \"shape\");" % n,
            "  " + asm([insn(t, k, n, n + 1, k) for k in range(n)], C, ['"v"(s)', '"v"(x)']),
            "}"]


def elims(T, t):
    """In-place elimination of n columns by row K (FP64): one overload per column count.  The
    one-column form ends with the wait states its consumer (a DPP broadcast of the next
    pivot, outside the block) needs."""
    out = []
    for n in range(1, 8):
        cols = ", ".join("%s &a%d" % (T, j) for j in range(n))
        outs = ['"+&v"(a%d)' % j for j in range(n)]
        out += per_lane("elim", "int K", "%s, %s c" % (cols, T), "K < %d" % LANES,
                        lambda k: asm([insn(t, j, j, n, k) for j in range(n)], outs, ['"v"(c)'],
                                      '"s_nop 1\\n"' if n == 1 else ""))
    return out


def prods(T, t, n, m):
    """C += X Y in one block: n columns of a product with an inner sum of m terms."""
    C = ['"+&v"(C[%d])' % j for j in range(n)]
    Y = ['"v"(Y[%d])' % j for j in range(n)]
    X = ['"v"(X[%d])' % k for k in range(m)]
    return ["template <int LC, int LY, int LX>",
            "__device__ __forceinline__ void prod%dx%d(%s (&C)[LC], const %s (&Y)[LY], const %s (&X)[LX]) {" % (m, n, T, T, T),
            "  static_assert(LC >= %d && LY >= %d && LX >= %d, \"shape\");" % (n, n, m),
            "  " + asm([insn(t, j, n + j, 2 * n + k, k) for k in range(m) for j in range(n)], C, Y + X),
            "}"]


def prodts(T, t, n, m):
    """C += X Y^T in one block: n columns (rows of Y) with an inner sum of m terms."""
    C = ['"+&v"(C[%d])' % j for j in range(n)]
    Y = ['"v"(Y[%d])' % j for j in range(m)]
    X = ['"v"(X[%d])' % k for k in range(m)]
    return ["template <int LC, int LY, int LX>",
            "__device__ __forceinline__ void prodt%dx%d(%s (&C)[LC], const %s (&Y)[LY], const %s (&X)[LX]) {" % (m, n, T, T, T),
            "  static_assert(LC >= %d && LY >= %d && LX >= %d, \"shape\");" % (n, m, m),
            "  " + asm([insn(t, j, n + k, n + m + k, j) for k in range(m) for j in range(n)], C, Y + X),
            "}"]


def render():
    parts = []
    for n in (14, 7):
        parts.append("\n".join(vectors("double", "f64", n)))
    for m, n in ((14, 14), (14, 8), (14, 7), (14, 4), (7, 7)):
        parts.append("\n".join(prods("double", "f64", n, m)))
    for m, n in ((14, 14), (7, 14)):
        parts.append("\n".join(prodts("double", "f64", n, m)))
    parts.append("\n".join(elims("double", "f64")))
    return HEADER + "\n" + "\n\n".join(parts) + "\n" + FOOTER


def main(argv):
    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "dpp_asm.h")
    text = render()
    if len(argv) > 1 and argv[1] == "--check":
        return 0 if open(path).read() == text else 1
    with open(path, "w") as f:
        f.write(text)
    return 0


if __name__ == "__main__":
    sys.exit(main(sys.argv))
