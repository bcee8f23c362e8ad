"""GPU tests of the 28-state direct solve's workspace: it lives in blocks that the context holds
anyway, so a first call allocates nothing but its schedule, and the separators' rows fit where a
batch needs the most of them per knot (problems of five knots: three for five), in a context
that holds just that batch.  Solves by both methods take turns, since they share the blocks.

The reference is the exact KKT solution; tolerance 1e-6 norm-wise as for the method's other tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import kkt
from paper_2309_08079_amd import synth

pytestmark = pytest.mark.gpu


def rel(a, b):
    a, b = np.asarray(a, dtype=np.float64).ravel(), np.asarray(b, dtype=np.float64).ravel()
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def context(knots, batch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_08079_amd.mpcpcg import Context
    return Context(28, 14, max_total_knots=knots, max_batch=batch)


def test_first_call_allocates_no_workspace():
    from paper_2309_08079_amd.mpcpcg import stats_to_numpy, to_device
    d = to_device(synth.problem(20, nx=28, nu=14, seed=4))
    small = context(32, 1)  # (loads the kernels)
    small.mpcpcg_set_method("factor")
    small.mpcpcg_solve(d)
    c = context(1 << 15, 4096)
    c.mpcpcg_set_method("factor")
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    out = c.mpcpcg_solve(d)
    torch.cuda.synchronize()
    assert free - torch.cuda.mem_get_info()[0] < 16 << 20
    assert stats_to_numpy(out["stats"])["status"][0] == 0
    c.close()
    small.close()


@pytest.mark.parametrize("Ns", [[5] * 8, [5], [2] * 8, [1], [1, 1, 5, 1, 17, 2], [21, 5, 85]])
def test_context_that_holds_just_the_batch(Ns):
    from paper_2309_08079_amd.mpcpcg import stats_to_numpy, to_device
    probs = synth.batch(Ns, seed0=400 + sum(Ns), nx=28, nu=14, defects=True)
    packed, off = synth.pack(probs)
    d = to_device(packed)
    c = context(sum(Ns), len(Ns))
    for method in ("factor", "pcg", "factor"):
        c.mpcpcg_set_method(method)
        out = c.mpcpcg_solve_batched(d, off)
        torch.cuda.synchronize()
        assert (stats_to_numpy(out["stats"])["status"] == 0).all()
    for b, p in enumerate(probs):
        ex = kkt.kkt_solve(p)
        k0, k1 = off[b], off[b + 1]
        assert rel(out["lam"][k0:k1].cpu().numpy(), ex["lam"]) < 1e-6, b
        assert rel(out["dx"][k0:k1].cpu().numpy(), ex["dx"]) < 1e-6, b
        if k1 - k0 > 1:
            assert rel(out["du"][k0 - b:k1 - b - 1].cpu().numpy(), ex["du"]) < 1e-6, b
    c.close()
