"""GPU tests of the 14-state direct solve's workspace: batches that need the most separators (a
problem of 4^l + 1 knots has the most rows per knot on level l, one of a single knot one) solved in
contexts that hold just them, and what the workspace takes of the device's memory.

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
    c = Context(14, 7, max_total_knots=knots, max_batch=batch)
    c.mpcpcg_set_method("factor")
    return c


@pytest.mark.parametrize("Ns", [[1] * 5, [2] * 8, [5] * 8, [17] * 3, [129, 1, 1, 5], [5, 17, 65, 257, 1025, 1, 513], [520], [2049]])
def test_context_that_holds_just_the_batch(Ns):
    from paper_2309_08079_amd.mpcpcg import stats_to_numpy, to_device
    probs = synth.batch(Ns, seed0=300 + sum(Ns), defects=True)
    packed, off = synth.pack(probs)
    c = context(sum(Ns), len(Ns))
    out = c.mpcpcg_solve_batched(to_device(packed), off)
    one = c.mpcpcg_solve(to_device(probs[0]))
    torch.cuda.synchronize()
    assert (stats_to_numpy(out["stats"])["status"] == 0).all()
    for b, p in enumerate(probs):
        ex = kkt.kkt_solve(p)
        k0, k1 = off[b], off[b + 1]
        assert rel(out["lam"][k0:k1].cpu().numpy(), ex["lam"]) < 1e-6, b
        assert rel(out["dx"][k0:k1].cpu().numpy(), ex["dx"]) < 1e-6, b
        if k1 - k0 > 1:
            assert rel(out["du"][k0 - b:k1 - b - 1].cpu().numpy(), ex["du"]) < 1e-6, b
    assert rel(one["lam"].cpu().numpy(), kkt.kkt_solve(probs[0])["lam"]) < 1e-6
    c.close()


def test_memory_of_the_workspace():
    # 3.7 KB per knot for W, H and z, 5.9 KB per separator
    from paper_2309_08079_amd.mpcpcg import to_device
    d = to_device(synth.problem(20, seed=4))
    small = context(32, 1)  # (loads the kernels)
    small.mpcpcg_solve(d)
    K = 1 << 15
    c = context(K, 4096)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    c.mpcpcg_solve(d)
    torch.cuda.synchronize()
    assert free - torch.cuda.mem_get_info()[0] < 8192 * K
    c.close()
    small.close()
