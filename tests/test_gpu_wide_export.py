"""GPU test of the 28-state Schur export, whose blocks the preconditioner's kernels write straight to
the caller's arrays (two knots to a wave, an odd count leaves half a wave without one): every
element is written, also where a block does not exist, at any alignment of the arrays.
Tolerances as for the other formation tests (FP32 rounding of S and gamma, and of Phi^-1)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import ref as orc
from paper_2309_08079_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 33])
def test_every_element_is_written(N, shift):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_08079_amd.mpcpcg import Context, to_device
    p = synth.problem(N, nx=28, nu=14, seed=520 + N, defects=True)
    buf = [torch.full((n + 2,), float("nan"), device="cuda") for n in (N * 3 * 784, N * 3 * 784, N * 28)]
    out = [b[shift:shift + b.numel() - 2].view(*s) for b, s in zip(buf, ((N, 3, 28, 28), (N, 3, 28, 28), (N, 28)))]
    c = Context(28, 14, max_total_knots=64, max_batch=1)
    c.mpcpcg_form_schur(to_device(p), out=out)
    torch.cuda.synchronize()
    c.close()
    for got, want, tol in zip(out, orc.form(p), (2e-7, 2e-6, 2e-7)):
        got = got.cpu().numpy().astype(np.float64)
        for b in range(N):
            assert np.linalg.norm(got[b] - want[b]) < tol * np.linalg.norm(want[b]), b
        if got.ndim == 4:
            assert not got[0, 0].any() and not got[-1, 2].any()
    for b in buf:  # nothing beside them is
        assert torch.isnan(b[:shift]).all() and torch.isnan(b[b.numel() - 2 + shift:]).all()
