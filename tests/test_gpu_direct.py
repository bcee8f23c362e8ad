"""GPU tests of the direct solves: of the 14-state one at the sizes where its split can go wrong: horizons
around a whole chunk (4 knots), around the separators that fit LDS (32, so 128 knots), and
around one, two and three levels of separators (512, 2048 knots), alone and in one ragged
batch, and the adjoint with every loss gradient given and with none but dL/dlambda.

The reference is the exact KKT solution (oracle/kkt.py).  Tolerances: lambda, dx, du 1e-6
norm-wise (kappa(S) ~ 3e3 times FP64 rounding, plus 6e-8 of the FP32 outputs), gradients
1e-5, as for the method's other tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import kkt
from paper_2309_08079_amd import synth

pytestmark = pytest.mark.gpu


def rel(a, b):
    a = np.asarray(a, dtype=np.float64).ravel()
    b = np.asarray(b, dtype=np.float64).ravel()
    nb = np.linalg.norm(b)
    return np.linalg.norm(a - b) / (nb if nb > 0 else 1.0)


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_08079_amd.mpcpcg import Context
    c = Context(14, 7, max_total_knots=1 << 13, max_batch=32)
    c.mpcpcg_set_method("factor")
    yield c
    c.close()


def dev(p):
    from paper_2309_08079_amd.mpcpcg import to_device
    return to_device(p)


def status(t):
    from paper_2309_08079_amd.mpcpcg import stats_to_numpy
    return stats_to_numpy(t)["status"]


@pytest.mark.parametrize("N", [4, 5, 8, 9, 127, 128, 129, 511, 513, 2047, 2049])
def test_single_at_the_edges_of_chunks_and_levels(ctx, N):
    p = synth.problem(N, seed=9700 + N, defects=(N % 2 == 0))
    out = ctx.mpcpcg_solve(dev(p))
    torch.cuda.synchronize()
    assert (status(out["stats"]) == 0).all()
    ex = kkt.kkt_solve(p)
    for k in ("lam", "dx", "du"):
        assert rel(out[k].cpu().numpy(), ex[k]) < 1e-6, k


@pytest.mark.parametrize("Ns", [[1, 4, 5, 3, 8, 127, 128, 129, 6, 31], [600, 1, 513, 2, 140, 36]])
def test_ragged_batches_share_the_levels(ctx, Ns):
    # short problems pass through the levels that the longest one needs
    probs = synth.batch(Ns, seed0=9800, defects=True)
    packed, off = synth.pack(probs)
    out = ctx.mpcpcg_solve_batched(dev(packed), off)
    torch.cuda.synchronize()
    assert (status(out["stats"]) == 0).all()
    for b, p in enumerate(probs):
        ex = kkt.kkt_solve(p)
        k0, k1 = off[b], off[b + 1]
        assert rel(out["lam"][k0:k1].cpu().numpy(), ex["lam"]) < 1e-6, b
        assert rel(out["dx"][k0:k1].cpu().numpy(), ex["dx"]) < 1e-6, b
        if k1 - k0 > 1:
            assert rel(out["du"][k0 - b:k1 - b - 1].cpu().numpy(), ex["du"]) < 1e-6, b


@pytest.mark.parametrize("losses", [False, True])
def test_adjoint_with_and_without_primal_loss_gradients(ctx, losses):
    Ns = [1, 5, 130, 9]
    probs = synth.batch(Ns, seed0=9900)
    packed, off = synth.pack(probs)
    d = dev(packed)
    if not losses:
        d.pop("e")  # no defects array at all (the draws are zero)
    fwd = ctx.mpcpcg_solve_batched(d, off)
    rng = np.random.default_rng(5)
    gl = rng.standard_normal(fwd["lam"].shape)
    gx = rng.standard_normal(fwd["dx"].shape) if losses else None
    gu = rng.standard_normal(fwd["du"].shape) if losses else None
    t = lambda v: None if v is None else torch.from_numpy(v.astype(np.float32)).cuda()
    g = ctx.mpcpcg_backward(d, off, fwd, t(gl), t(gx), t(gu))
    torch.cuda.synchronize()
    assert (status(g["stats"]) == 0).all()
    f32 = lambda v, a, b: None if v is None else v.astype(np.float32).astype(np.float64)[a:b]
    for b, p in enumerate(probs):
        k0, k1 = off[b], off[b + 1]
        c0, c1 = k0 - b, k1 - b - 1
        ref = kkt.adjoint_dense(p, f32(gl, k0, k1), f32(gx, k0, k1), f32(gu, c0, c1))
        for k, a, z in (("dQ", k0, k1), ("dq", k0, k1), ("dR", c0, c1), ("dA", c0, c1), ("dB", c0, c1), ("dr", c0, c1), ("de", c0, c1)):
            if z > a:
                assert rel(g[k][a:z].cpu().numpy(), ref[k]) < 1e-5, (b, k)
        assert rel(g["dx0"][b].cpu().numpy(), ref["dx0"]) < 1e-5, b


# ---------------------------------------------------------------- 28 states
# The two-arm path's chunks are of 4 rows on every level, two knots to a wave (an odd count
# leaves half a wave without a knot); the last row of each problem is solved by itself.
@pytest.fixture(scope="module")
def wide():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_08079_amd.mpcpcg import Context
    c = Context(28, 14, max_total_knots=1 << 10, max_batch=16)
    c.mpcpcg_set_method("factor")
    yield c
    c.close()


@pytest.mark.parametrize("Ns", [[1], [2], [3], [4], [5], [16], [17], [64], [65], [257], [1, 4, 5, 3, 2, 16, 17, 66, 9]])
def test_two_arm_at_the_edges_of_chunks_and_levels(wide, Ns):
    probs = synth.batch(Ns, seed0=9950 + len(Ns) + Ns[0], nx=28, nu=14, defects=True)
    packed, off = synth.pack(probs)
    d = dev(packed)
    fwd = wide.mpcpcg_solve_batched(d, off)
    rng = np.random.default_rng(6)
    gl, gx, gu = (rng.standard_normal(fwd[k].shape).astype(np.float32) for k in ("lam", "dx", "du"))
    g = wide.mpcpcg_backward(d, off, fwd, *(torch.from_numpy(v).cuda() for v in (gl, gx, gu)))
    torch.cuda.synchronize()
    assert (status(fwd["stats"]) == 0).all() and (status(g["stats"]) == 0).all()
    gl, gx, gu = (v.astype(np.float64) for v in (gl, gx, gu))
    for b, p in enumerate(probs):
        k0, k1 = off[b], off[b + 1]
        c0, c1 = k0 - b, k1 - b - 1
        ex = kkt.kkt_solve(p)
        for k, a, z in (("lam", k0, k1), ("dx", k0, k1), ("du", c0, c1)):
            if z > a:
                assert rel(fwd[k][a:z].cpu().numpy(), ex[k]) < 1e-6, (b, k)
        if k1 - k0 > 66:
            continue  # (the dense adjoint of the oracle is cubic)
        ref = kkt.adjoint_dense(p, gl[k0:k1], gx[k0:k1], gu[c0:c1])
        for k, a, z in (("dQ", k0, k1), ("dq", k0, k1), ("dR", c0, c1), ("dA", c0, c1), ("dB", c0, c1), ("dr", c0, c1), ("de", c0, c1)):
            if z > a:
                assert rel(g[k][a:z].cpu().numpy(), ref[k]) < 1e-5, (b, k)
        assert rel(g["dx0"][b].cpu().numpy(), ref["dx0"]) < 1e-5, b
