"""GPU tests of the 28-state PCG at the edges of its split: four knots (waves) to a workgroup,
so one part, one part and a knot, whole and ragged last parts, and more parts than one poll of
64 covers; cold and warm; and on one XCD (barriers through its L2) against device scope, which
must agree bit for bit.

Tolerances as for the method's other tests: lambda within 1e-5 of the oracle's PCG iterate, the
count of iterations within two or a tenth."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import ref as orc
from paper_2309_08079_amd import synth

pytestmark = pytest.mark.gpu
EPS = 1e-6


@pytest.mark.parametrize("warm", [False, True])
@pytest.mark.parametrize("N", [1, 3, 4, 5, 8, 9, 260])
def test_parts_of_a_gang(N, warm):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_08079_amd.mpcpcg import Context, stats_to_numpy, to_device
    p = synth.problem(N, nx=28, nu=14, seed=640 + N, defects=True)
    lam0 = 0.1 * np.random.default_rng(N).standard_normal((N, 28)).astype(np.float32) if warm else None
    got = []
    for pin in (1, 0):
        c = Context(28, 14, max_total_knots=512, max_batch=2)
        c.mpcpcg_set_method("pcg")
        c.mpcpcg_set_xcd_pinning(pin)
        out = c.mpcpcg_solve(to_device(p), eps=EPS, lam0=torch.from_numpy(lam0).cuda() if warm else None)
        torch.cuda.synchronize()
        got.append((out["lam"].cpu().numpy().reshape(N, 28), stats_to_numpy(out["stats"])))
        c.close()
    ref = orc.solve(p, eps=EPS, lam0=lam0.astype(np.float64) if warm else None)
    lam, st = got[0]
    assert (st["status"] == 0).all()
    assert abs(int(st["iters"][0]) - ref["iters"]) <= max(2, ref["iters"] // 10)
    assert np.linalg.norm(lam - ref["lam"]) < 1e-5 * np.linalg.norm(ref["lam"])
    assert np.array_equal(lam, got[1][0]) and st["iters"][0] == got[1][1]["iters"][0]
