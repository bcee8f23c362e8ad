"""GPU test of the stopping rule where it cannot decide: with eps infinite and a right-hand side
of zeros the threshold eps^2 gamma^T Phi^-1 gamma is not a number, no test against it holds, and
the solve ends at its first division (BREAKDOWN), as the oracle's loop does."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import ref as orc
from paper_2309_08079_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nu", [(14, 7), (28, 14)])
@pytest.mark.parametrize("N", [1, 16, 40])
def test_threshold_that_is_not_a_number(nx, nu, N):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_08079_amd.mpcpcg import Context, stats_to_numpy, to_device
    p = synth.problem(N, nx=nx, nu=nu, seed=90 + N)
    for k in ("q", "r", "x0", "e"):
        p[k] = np.zeros_like(p[k])
    want = orc.solve(p, eps=float("inf"))
    c = Context(nx, nu, max_total_knots=64, max_batch=2)
    out = c.mpcpcg_solve(to_device(p), eps=float("inf"))
    torch.cuda.synchronize()
    st = stats_to_numpy(out["stats"])[0]
    c.close()
    assert st["status"] == want["status"]
