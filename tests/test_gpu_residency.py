"""GPU tests of the rule that picks the 14-state kernel's form: launches whose workgroups all fit
at two waves per SIMD (two 16-knot workgroups per compute unit, 512 on the device) keep Phi^-1
in registers, larger ones in LDS.  The two forms do the same operations in the same order, so
a problem's results must not depend on the size of the batch around it: bit for bit, forward,
adjoint and adjoint from the kept factors, on one XCD per gang and from the global queue, on
both sides of the line and for one problem by itself."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2309_08079_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pin", [1, 0])
def test_results_do_not_depend_on_the_batch_around_a_problem(pin):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_08079_amd.mpcpcg import Context, to_device
    probs = [synth.problem(n, seed=8100 + n, defects=True) for n in (40, 16, 17)]  # 3 + 1 + 2 parts
    c = Context(14, 7, max_total_knots=1 << 13, max_batch=300)
    c.mpcpcg_set_xcd_pinning(pin)

    def run(times):
        packed, off = synth.pack(probs * times)
        d = to_device(packed)
        rec = c.factor_record(int(off[-1]), "cuda")
        f = c.mpcpcg_solve_batched(d, off, factors=rec)
        g = c.mpcpcg_backward(d, off, f, 2 * f["lam"])
        k = c.mpcpcg_backward(d, off, f, 2 * f["lam"], factors=rec)
        torch.cuda.synchronize()
        n, m = off[3], off[3] - 3
        return [f["lam"][:n], f["dx"][:n], f["du"][:m], f["stats"][:3], g["dQ"][:n], g["dA"][:m], g["stats"][:3],
                k["dQ"][:n], k["dA"][:m], k["stats"][:3]], [f["lam"][-n:], g["dQ"][-n:], k["dQ"][-n:]]

    first, last = run(1)
    assert torch.equal(first[4], first[7])  # the adjoint with and without the kept factors
    for times in (85, 86):  # 510 and 516 workgroups
        a, z = run(times)
        for x, y in zip(a, first):
            assert torch.equal(x, y), times
        for x, y in zip(z, last):
            assert torch.equal(x, y), times
    for i, p in enumerate(probs):  # alone
        out = c.mpcpcg_solve(to_device(p))
        torch.cuda.synchronize()
        n0 = sum(q["q"].shape[0] for q in probs[:i])
        assert torch.equal(out["lam"], first[0][n0:n0 + p["q"].shape[0]]), i
    c.close()
