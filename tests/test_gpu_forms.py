"""GPU tests of the 14-state kernel's two-waves-per-SIMD form, which launches of one-part problems
take while all their workgroups are resident (two 16-knot workgroups per compute unit, 512 on
the device, 64 per XCD list).  Both forms do the same operations in the same order, so the results
must not depend on the size of the batch, bit for bit: forward, adjoint and adjoint from the kept factors,
per XCD and from the global queue, on both sides of the line and beside a longer problem, which
takes the launch to the other form; and single solves on four streams, whose gangs fill the XCD
they share."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2309_08079_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pin", [1, 0])
def test_one_part_problems_on_both_sides_of_the_line(pin):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_08079_amd.mpcpcg import Context, to_device
    probs = [synth.problem(n, seed=8200 + n, defects=True) for n in (16, 1, 9, 4)]
    c = Context(14, 7, max_total_knots=1 << 13, max_batch=600)
    c.mpcpcg_set_xcd_pinning(pin)
    n, m = 30, 26  # knots and controls of the four

    def run(batch):
        packed, off = synth.pack(batch)
        d = to_device(packed)
        rec = c.factor_record(int(off[-1]), "cuda")
        f = c.mpcpcg_solve_batched(d, off, factors=rec)
        g = c.mpcpcg_backward(d, off, f, 2 * f["lam"])
        k = c.mpcpcg_backward(d, off, f, 2 * f["lam"], factors=rec)
        torch.cuda.synchronize()
        return [f["lam"][:n], f["dx"][:n], f["du"][:m], f["stats"][:4], g["dQ"][:n], g["dA"][:m], g["stats"][:4],
                k["dQ"][:n], k["dA"][:m], k["stats"][:4]]

    first = run(probs)
    assert (first[3][:, 1] == 0).all() and (first[6][:, 1] == 0).all()
    assert torch.equal(first[4], first[7])  # the adjoint with and without the kept factors
    long = synth.problem(40, seed=8300)
    for batch in (probs * 127 + probs[:3], probs * 128, probs * 128 + probs[:1], probs * 129, probs + [long]):
        for x, y in zip(run(batch), first):
            assert torch.equal(x, y), len(batch)
    c.close()


def test_single_solves_on_four_streams_find_their_places():
    # 32 + 32 + 16 + 16 parts, the 96 places of the XCD that single solves share: every solve ends
    # and has the bits it has alone
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_08079_amd.mpcpcg import Context, to_device
    Ns = [512, 512, 256, 256]
    ctx = [Context(14, 7, max_total_knots=n, max_batch=1) for n in Ns]
    d = [to_device(synth.problem(n, seed=8400 + i)) for i, n in enumerate(Ns)]
    alone = []
    for c, p in zip(ctx, d):
        o = c.mpcpcg_solve(p)
        torch.cuda.synchronize()
        alone.append({k: v.clone() for k, v in o.items()})
    streams = [torch.cuda.Stream() for _ in Ns]
    outs = [[] for _ in Ns]
    torch.cuda.synchronize()
    for _ in range(10):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                outs[i].append(ctx[i].mpcpcg_solve(d[i]))
    torch.cuda.synchronize()
    for i, want in enumerate(alone):
        assert want["stats"][0, 1] == 0
        for o in outs[i]:
            for k in ("lam", "dx", "du", "stats"):
                assert torch.equal(o[k], want[k]), (i, k)
    for c in ctx:
        c.close()
