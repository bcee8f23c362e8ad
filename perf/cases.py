"""The work a user of libmpcpcg has it do, as cases that can be timed and checked.

``listed()`` names the cases, ``draw(rng)`` gives more of the same ranges, ``prepare`` makes
what a program holds before the call (problem data on the GPU, a context, output buffers),
``run`` is one pass through the public entry points, ``work`` the bytes and operations of a
pass, and ``exact`` its result in 64 bits from the plain definitions.

Inputs follow the recipe of ``paper_2309_08079_amd.synth`` (Kuka-shaped linear-quadratic
problems, pendulum-chain trajectories), drawn on the GPU from the seed.
"""
import random

import numpy as np
import torch

from paper_2309_08079_amd import Context, MPCPCGFunction

DEV = "cuda"
EPS = 1e-6


def listed():
    return [
        # building the Schur system and its preconditioner for a caller's own solver
        dict(name="schur_n128", kind="schur", nx=14, n=128),
        # one short solve, cold: the smallest size the paper measures
        dict(name="solve_n32", kind="solve", nx=14, n=32, defects=False),
        # one long solve, cold: the largest size the paper measures
        dict(name="solve_n512", kind="solve", nx=14, n=512, defects=False),
        # one step of a receding-horizon controller: warm-started from the last step's
        # multipliers, stopped by the paper's absolute rule
        dict(name="warm_n128", kind="warm", nx=14, n=128, defects=True),
        # many planners at once, horizons from the paper's sizes
        dict(name="mixed_batch", kind="batch", nx=14, b=256, lo=32, hi=512, spread="pow2", method="pcg", defects=False),
        # differentiable MPC as a layer: forward and backward through the autograd function
        dict(name="gradient_layer", kind="layer", nx=14, b=64, lo=128, hi=128, spread="same", defects=True),
        # training throughput, forward (keeping its preconditioner) and adjoint of a large batch
        dict(name="train_256x512", kind="train", nx=14, b=256, lo=512, hi=512, spread="same", method="pcg", keep=True, q_lo=1.0, q_hi=10.0),
        # the direct method on a ragged batch, forward and adjoint
        dict(name="direct_ragged", kind="train", nx=14, b=256, lo=17, hi=500, spread="int", method="factor", keep=False, q_lo=1.0, q_hi=10.0),
        # two arms (28 states), the default iterative method, forward and adjoint
        dict(name="two_arm_pcg", kind="train", nx=28, b=32, lo=64, hi=256, spread="int", method="pcg", keep=False, q_lo=1.0, q_hi=10.0),
        # two arms, badly scaled costs, the method the library picks: forward and adjoint
        dict(name="two_arm_auto", kind="train", nx=28, b=32, lo=64, hi=256, spread="int", method="auto", keep=False, q_lo=1e-2, q_hi=1e2),
        # one robot's control step (linearise, solve, line search) as one call
        dict(name="control_n128", kind="control", nx=14, b=1, n=128, method="factor", sqp=1),
        # control steps of many robots as one call
        dict(name="control_256x128", kind="control", nx=14, b=256, n=128, method="auto", sqp=1),
    ]


KNOTS = 131072  # the most knots of a 14-state case (the largest listed one's)


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(["schur", "solve", "solve", "warm", "batch", "layer", "train", "direct", "two_pcg", "two_auto", "control", "control"])
    if kind == "schur":
        return dict(kind="schur", nx=rng.choice([14, 14, 28]), n=_log_int(rng, 2, 290))
    if kind == "solve":
        return dict(kind="solve", nx=14, n=_log_int(rng, 2, 1024), defects=rng.random() < 0.5)
    if kind == "warm":
        return dict(kind="warm", nx=14, n=_log_int(rng, 8, 512), defects=rng.random() < 0.5)
    if kind == "control":
        b = rng.choice([1, 1, _log_int(rng, 2, 256)])
        return dict(kind="control", nx=14, b=b, n=_log_int(rng, 8, min(512, KNOTS // (4 * b))),
                    method="factor" if b == 1 else "auto", sqp=rng.choice([1, 2]))
    hseed = rng.randrange(1 << 20)
    spread = rng.choice(["same", "int", "pow2"])
    if kind in ("two_pcg", "two_auto"):
        hi = rng.randint(16, 256)
        wide = kind == "two_auto"
        return dict(kind="train", nx=28, b=_log_int(rng, 1, 32), lo=max(2, hi // 4), hi=hi, spread="same" if spread == "pow2" else spread,
                    method="auto" if wide else "pcg", keep=False, q_lo=1e-2 if wide else 1.0, q_hi=1e2 if wide else 10.0, hseed=hseed)
    b = _log_int(rng, 1, 256)
    hi = 512 if spread == "pow2" else _log_int(rng, 8, 512)
    lo = hi if spread == "same" else (32 if spread == "pow2" else max(2, hi // 16))
    c = dict(nx=14, b=b, lo=lo, hi=hi, spread=spread, hseed=hseed)
    if kind == "batch":
        return dict(c, kind="batch", method=rng.choice(["pcg", "pcg", "auto"]), defects=rng.random() < 0.5)
    if kind == "layer":
        return dict(c, kind="layer", b=min(b, 64), defects=rng.random() < 0.5)
    if kind == "train":
        return dict(c, kind="train", method="pcg", keep=rng.random() < 0.7, q_lo=1.0, q_hi=10.0)
    return dict(c, kind="train", method="factor", keep=False, q_lo=1.0, q_hi=10.0)


# ---- sizes ---------------------------------------------------------------------------------


def _horizons(case):
    if "lo" not in case:
        return [case["n"]] * case.get("b", 1)
    g = random.Random(case.get("hseed", 3000))
    if case["spread"] == "same":
        return [case["hi"]] * case["b"]
    if case["spread"] == "pow2":
        return [g.choice([n for n in (32, 64, 128, 256, 512) if case["lo"] <= n <= case["hi"]]) for _ in range(case["b"])]
    return [g.randint(case["lo"], case["hi"]) for _ in range(case["b"])]


def _offsets(Ns):
    return np.concatenate([[0], np.cumsum(Ns)]).astype(np.int64)


# ---- inputs --------------------------------------------------------------------------------


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _costs(g, K, M, nx, nu, q_lo, q_hi, r_lo, r_hi):
    f = dict(generator=g, device=DEV, dtype=torch.float64)
    W = torch.randn(K, nx, 4, **f)
    Q = torch.zeros(K, nx, nx, device=DEV, dtype=torch.float64)
    for j in range(4):
        Q += 0.1 * W[:, :, j, None] * W[:, None, :, j]
    Q.diagonal(dim1=1, dim2=2).add_(q_lo + (q_hi - q_lo) * torch.rand(K, nx, **f))
    R = torch.zeros(M, nu, nu, device=DEV, dtype=torch.float64)
    R.diagonal(dim1=1, dim2=2).add_(r_lo + (r_hi - r_lo) * torch.rand(M, nu, **f))
    return Q, R


def _problem(case, seed):
    """A packed batch of linear-quadratic problems (synth.problem's recipe)."""
    Ns = _horizons(case)
    nx, B = case["nx"], len(Ns)
    nu, K = nx // 2, sum(Ns)
    M = K - B
    g = _gen(seed)
    f = dict(generator=g, device=DEV, dtype=torch.float64)
    Q, R = _costs(g, K, M, nx, nu, case.get("q_lo", 1.0), case.get("q_hi", 10.0), 0.1, 1.0)
    p = dict(Q=Q, R=R, A=torch.eye(nx, device=DEV, dtype=torch.float64) + 0.01 * torch.randn(M, nx, nx, **f),
             B=0.01 * torch.randn(M, nx, nu, **f), q=torch.randn(K, nx, **f), r=torch.randn(M, nu, **f),
             x0=torch.randn(B, nx, **f))
    e = 0.01 * torch.randn(M, nx, **f)
    if case.get("defects"):
        p["e"] = e
    return {k: v.float().contiguous() for k, v in p.items()}


def _model():
    g = torch.Generator().manual_seed(10000)
    return dict(h=float(np.float32(0.01)), damping=0.5, coupling=2.0, gravity=(5.0 + 10.0 * torch.rand(7, generator=g)).to(DEV))


def _trajectory(case, seed):
    """Packed pendulum-chain trajectories (synth.trajectory's recipe): a guess that violates
    the dynamics, a measured state and a goal away from it."""
    B, N, nx = case["b"], case["n"], case["nx"]
    nu = nx // 2
    g = _gen(seed)
    f = dict(generator=g, device=DEV, dtype=torch.float64)
    xi = torch.cat([2 * torch.rand(B, nu, **f) - 1, 0.5 * torch.randn(B, nu, **f)], 1)
    goal = torch.cat([2 * torch.rand(B, nu, **f) - 1, torch.zeros(B, nu, device=DEV, dtype=torch.float64)], 1)
    t = (torch.arange(N, device=DEV, dtype=torch.float64) / max(N - 1, 1))[None, :, None]
    X = (1 - t) * xi[:, None] + t * goal[:, None] + 0.3 * torch.randn(B, N, nx, **f)
    U = 0.5 * torch.randn(B * (N - 1), nu, **f)
    Q, R = _costs(g, B * N, B * (N - 1), nx, nu, 1.0, 10.0, 1e-3, 1e-2)
    d = dict(X=X.reshape(B * N, nx), U=U, x_init=xi, xref=goal[:, None].expand(B, N, nx).reshape(B * N, nx), Q=Q, R=R)
    return {k: v.float().contiguous() for k, v in d.items()}


def _warm_lambda(case, seed, p):
    """The last step's multipliers: those of the same horizon with the state where it was."""
    prev = dict(p, x0=(p["x0"].double() + 0.05 * torch.randn(p["x0"].shape, generator=_gen(seed + 77), device=DEV, dtype=torch.float64)).float())
    lam, _, _ = _solve64(_padded(prev, _horizons(case)))
    return lam.reshape(-1, case["nx"]).float().to(DEV).contiguous()


def prepare(case, seed):
    Ns = _horizons(case)
    off = _offsets(Ns)
    K, B, nx = int(off[-1]), len(Ns), case["nx"]
    M, nu, kind = K - B, nx // 2, case["kind"]
    new = lambda *s, dtype=torch.float32: torch.zeros(s, device=DEV, dtype=dtype)  # noqa: E731
    ctx = Context(nx, nu, max_total_knots=K, max_batch=B)
    ctx.mpcpcg_set_method(case.get("method", "pcg"))
    s = dict(kind=kind, ctx=ctx, off=off, sqp=case.get("sqp", 1))
    if kind == "control":
        s.update(model=_model(), traj=_trajectory(case, seed), lam=new(K, nx), X=new(K, nx), U=new(M, nu),
                 out=dict(merit=new(B, 9, dtype=torch.float64), choice=new(B, dtype=torch.int32), stats=new(B, 4, dtype=torch.int32)))
        return s
    p = s["p"] = _problem(case, seed)
    if kind == "schur":
        s["out"] = (new(K, 3, nx, nx), new(K, 3, nx, nx), new(K, nx))
        return s
    if kind == "layer":
        for k in p:
            p[k].requires_grad_(True)
        return s
    s["out"] = dict(lam=new(K, nx), dx=new(K, nx), du=new(M, nu), stats=new(B, 4, dtype=torch.int32))
    if kind == "warm":
        s["lam0"] = _warm_lambda(case, seed, p)
    if kind == "train":
        s["rec"] = ctx.factor_record(K, DEV) if case["keep"] else None
        s["grad"] = dict(dQ=new(K, nx, nx), dR=new(M, nu, nu), dA=new(M, nx, nx), dB=new(M, nx, nu), dq=new(K, nx), dr=new(M, nu),
                         dx0=new(B, nx), de=new(M, nx), dgamma=new(K, nx), stats=new(B, 4, dtype=torch.int32))
    return s


# ---- one pass ------------------------------------------------------------------------------
# The solver's stats come back as the outcome of each problem (its status).  The iteration
# count and the exit ratio beside it describe the Krylov path, which a different order of
# the same sums may lengthen or shorten by one, and the line search's merits are scores of
# steps already rounded to 32 bits: neither is a result of the pass.


def run(s):
    kind, ctx = s["kind"], s["ctx"]
    if kind == "schur":
        S, P, g = ctx.mpcpcg_form_schur(s["p"], out=s["out"])
        return dict(S=S, Pinv=P, gamma=g)
    if kind == "solve":
        f = ctx.mpcpcg_solve(s["p"], eps=EPS, out=s["out"])
    elif kind == "warm":
        f = ctx.mpcpcg_solve(s["p"], eps=1e-5, lam0=s["lam0"], stop="absolute", out=s["out"])
    elif kind == "batch":
        f = ctx.mpcpcg_solve_batched(s["p"], s["off"], eps=EPS, out=s["out"])
    elif kind == "train":
        f = ctx.mpcpcg_solve_batched(s["p"], s["off"], eps=EPS, out=s["out"], factors=s["rec"])
        g = ctx.mpcpcg_backward(s["p"], s["off"], f, 2 * f["lam"], eps=EPS, out=s["grad"], factors=s["rec"])
        return dict(lam=f["lam"], dx=f["dx"], du=f["du"], grad={k: v for k, v in g.items() if k != "stats"},
                    status=[f["stats"][:, 1], g["stats"][:, 1]])
    elif kind == "layer":
        p = s["p"]
        lam, dx, du = MPCPCGFunction.apply(ctx, s["off"], EPS, p["Q"], p["R"], p["A"], p["B"], p["q"], p["r"], p["x0"], p.get("e"))
        g = torch.autograd.grad(lam.square().sum(), list(p.values()))
        return dict(lam=lam.detach(), dx=dx.detach(), du=du.detach(), grad={"d" + k: v for k, v in zip(p, g)})
    else:
        o = ctx.mpcpcg_control_step(s["model"], s["traj"], s["off"], s["lam"], s["X"], s["U"], sqp_iters=s["sqp"], mu=1.0, out=s["out"])
        return dict(X=s["X"], U=s["U"], lam=s["lam"], choice=o["choice"], status=o["stats"][:, 1])
    return dict(lam=f["lam"], dx=f["dx"], du=f["du"], status=f["stats"][:, 1])


# ---- what a pass cannot do without ---------------------------------------------------------


def work(case):
    """Inputs read once, outputs written once; multiply-adds of the formation, of ~105 PCG
    iterations (~50 warm) or one block factorisation, and of the primal step and gradients."""
    Ns = _horizons(case)
    K, B, nx, kind = sum(Ns), len(Ns), case["nx"], case["kind"]
    nu, M = nx // 2, K - B
    data = K * (nx * nx + nx) + M * (nu * nu + nx * nx + nx * nu + nu) + B * nx
    if case.get("defects"):
        data += M * nx
    sol = 2 * K * nx + M * nu
    n3 = nx ** 3
    form = 2 * (n3 + nu ** 3 + 2 * n3 + 1.5 * nx * nx * nu)   # Q^-1, R^-1, A Q^-1 A^T, B R^-1 B^T
    stair = 2 * (n3 + 2 * n3)                                  # D^-1 and the two off-diagonal blocks
    step = 2 * (2 * nx * nx + nx * nu + nu * nu)
    it = 2 * 6 * nx * nx + 10 * nx
    factor = 2 * (2.4 * n3 + 4 * nx * nx)
    grad = 2 * (2 * nx * nx + 2 * nx * nx + 2 * nx * nu + 2 * nu * nu)
    pcg = kind in ("solve", "warm", "layer") or case.get("method") == "pcg"
    solve = stair + 105 * it if pcg else factor
    if kind == "schur":
        return dict(bytes=4.0 * (data + 6 * K * nx * nx + K * nx), flops=float(K * (form + stair)))
    if kind == "warm":
        return dict(bytes=4.0 * (data + sol + K * nx), flops=float(K * (form + stair + 50 * it + step)))
    if kind in ("solve", "batch"):
        return dict(bytes=4.0 * (data + sol), flops=float(K * (form + solve + step)))
    if kind in ("train", "layer"):
        grads = K * (nx * nx + nx) + M * (nu * nu + nx * nx + nx * nu + nu) + B * nx
        if kind == "train" or case.get("defects"):
            grads += M * nx
        grads += K * nx if kind == "train" else 0
        return dict(bytes=4.0 * (data + sol + grads), flops=float(K * (form + solve + step + (solve - (stair if pcg else 0)) + step + grad)))
    weights = K * nx * nx + M * nu * nu
    line = 2 * nx * nx + 9 * 40 * nu
    return dict(bytes=4.0 * (weights + 2 * K * nx + M * nu + B * nx + 2 * K * nx + M * nu),
                flops=float(case["sqp"] * K * (form + factor + step + line)))


# ---- the same results in 64 bits -----------------------------------------------------------


def _padded(p, Ns):
    """float64 CPU arrays [batch, longest horizon, ...]: knots past a problem's horizon get
    identity costs and no dynamics, so that they stay apart from it."""
    off, B, N = _offsets(Ns), len(Ns), max(Ns)
    nx = p["q"].shape[1]
    nu = p["r"].shape[1]
    c = {k: v.detach().double().cpu() for k, v in p.items()}
    if "e" not in c:
        c["e"] = torch.zeros(c["r"].shape[0], nx, dtype=torch.float64)
    kn = torch.cat([torch.arange(n) + b * N for b, n in enumerate(Ns)])
    ct = torch.cat([torch.arange(n - 1) + b * N for b, n in enumerate(Ns)])

    def place(v, at, fill=None):
        out = torch.zeros((B * N,) + v.shape[1:], dtype=torch.float64)
        if fill is not None:
            out += torch.eye(fill, dtype=torch.float64)
        out[at] = v
        return out.reshape((B, N) + v.shape[1:])

    d = dict(Q=place(c["Q"], kn, nx), q=place(c["q"], kn), R=place(c["R"], ct, nu), A=place(c["A"], ct), B=place(c["B"], ct),
             r=place(c["r"], ct), e=place(c["e"], ct), x0=c["x0"].reshape(B, nx), kn=kn, ct=ct)
    d["Qi"], d["Ri"] = torch.linalg.inv(d["Q"]), torch.linalg.inv(d["R"])
    return d


def _mv(A, x):
    return (A @ x[..., None])[..., 0]


def _tmv(A, x):
    return _mv(A.transpose(-1, -2).contiguous(), x)


def _blocks64(d):
    """S_bb and S_{b,b+1} of C G^-1 C^T."""
    A, Bm, Qi, Ri = d["A"], d["B"], d["Qi"], d["Ri"]
    D = Qi.clone()
    D[:, 1:] += (A @ Qi @ A.transpose(-1, -2) + Bm @ Ri @ Bm.transpose(-1, -2))[:, :-1]
    return D, -(Qi @ A.transpose(-1, -2))


def _rhs64(d, gx, gu, top):
    """C G^-1 [gx; gu] + top."""
    qq, rr = _mv(d["Qi"], gx), _mv(d["Ri"], gu)
    y = qq + top
    y[:, 1:] -= (_mv(d["A"], qq) + _mv(d["B"], rr))[:, :-1]
    return y


def _tri64(d, y):
    """The block-tridiagonal solve, knot by knot."""
    D, U = d["S"] if "S" in d else d.setdefault("S", _blocks64(d))
    N = D.shape[1]
    Us, ys = [], []
    for k in range(N):
        Dk, yk = D[:, k], y[:, k]
        if k:
            L = U[:, k - 1].transpose(-1, -2)
            Dk, yk = Dk - L @ Us[-1], yk - _mv(L, ys[-1])
        X = torch.linalg.solve(Dk, torch.cat([U[:, k], yk[..., None]], -1))
        Us.append(X[..., :-1])
        ys.append(X[..., -1])
    x = [ys[-1]]
    for k in range(N - 2, -1, -1):
        x.append(ys[k] - _mv(Us[k], x[-1]))
    return torch.stack(x[::-1], 1)


def _primal64(d, lam, gx, gu):
    nxt = torch.zeros_like(lam)
    nxt[:, :-1] = lam[:, 1:]
    return -_mv(d["Qi"], gx - lam + _tmv(d["A"], nxt)), -_mv(d["Ri"], gu + _tmv(d["B"], nxt))


def _solve64(d):
    top = torch.zeros_like(d["q"])
    top[:, 0] = d["x0"]
    top[:, 1:] -= d["e"][:, :-1]
    lam = _tri64(d, _rhs64(d, d["q"], d["r"], top))
    return (lam, *_primal64(d, lam, d["q"], d["r"]))


def _knots(d, v):
    return v.reshape((-1,) + v.shape[2:])[d["kn"]]


def _ctrls(d, v):
    return v.reshape((-1,) + v.shape[2:])[d["ct"]]


def _grad64(d, lam, dx, du):
    """Adjoint of L = ||lambda||^2."""
    z, zu = torch.zeros_like(lam), torch.zeros_like(du)
    mu = _tri64(d, 2 * lam)
    nx_, nu_ = _primal64(d, mu, z, zu)
    outer = lambda a, b: a[..., :, None] * b[..., None, :]  # noqa: E731
    sym = lambda a, b: 0.5 * (outer(a, b) + outer(b, a))  # noqa: E731
    l1, m1 = torch.zeros_like(lam), torch.zeros_like(mu)
    l1[:, :-1], m1[:, :-1] = lam[:, 1:], mu[:, 1:]
    K, C = lambda v: _knots(d, v), lambda v: _ctrls(d, v)  # noqa: E731
    return dict(dQ=K(sym(nx_, dx)), dR=C(sym(nu_, du)), dA=C(outer(l1, nx_) + outer(m1, dx)), dB=C(outer(l1, nu_) + outer(m1, du)),
                dq=K(nx_), dr=C(nu_), dx0=mu[:, 0], de=C(-m1), dgamma=K(mu))


def _schur64(d):
    D, U = _blocks64(d)
    N, nx = D.shape[1], D.shape[2]
    S = torch.zeros(N, 3, nx, nx, dtype=torch.float64)
    S[:, 1] = D[0]
    S[:-1, 2] = U[0, :-1]
    S[1:, 0] = U[0, :-1].transpose(-1, -2)
    Di = torch.linalg.inv(D[0])
    P = torch.zeros_like(S)
    P[:, 1] = Di
    P[1:, 0] = -(Di[1:] @ S[1:, 0] @ Di[:-1])
    P[:-1, 2] = -(Di[:-1] @ S[:-1, 2] @ Di[1:])
    top = torch.zeros_like(d["q"])
    top[:, 0] = d["x0"]
    top[:, 1:] -= d["e"][:, :-1]
    return dict(S=S, Pinv=P, gamma=_rhs64(d, d["q"], d["r"], top)[0])


def _chain64(m, q, v, u):
    """Velocities and accelerations of the pendulum chain."""
    acc = u - m["g"] * torch.sin(q) - m["damping"] * v
    d = m["coupling"] * torch.sin(q[..., 1:] - q[..., :-1])
    acc[..., :-1] += d
    acc[..., 1:] -= d
    return acc


def _step64(m, x, u):
    nq = u.shape[-1]
    q, v = x[..., :nq], x[..., nq:]
    return torch.cat([q + m["h"] * v, v + m["h"] * _chain64(m, q, v, u)], -1)


def _control64(case, t):
    B, N, nx = case["b"], case["n"], case["nx"]
    nu = nx // 2
    mod = _model()
    m = dict(h=mod["h"], damping=mod["damping"], coupling=mod["coupling"], g=mod["gravity"].double().cpu())
    c = {k: v.double().cpu() for k, v in t.items()}
    X, U = c["X"].reshape(B, N, nx), c["U"].reshape(B, N - 1, nu)
    Q, R = c["Q"].reshape(B, N, nx, nx), c["R"].reshape(B, N - 1, nu, nu)
    xr, xi = c["xref"].reshape(B, N, nx), c["x_init"]
    viol = lambda X, U: ((X[:, 0] - xi).abs().sum(1) + (X[:, 1:] - _step64(m, X[:, :-1], U)).abs().sum((1, 2)))  # noqa: E731
    cost = lambda X, U: 0.5 * (((X - xr) * _mv(Q, X - xr)).sum((1, 2)) + (U * _mv(R, U)).sum((1, 2)))  # noqa: E731
    for _ in range(case["sqp"]):
        q = X[:, :-1, :nu]
        A = torch.zeros(B, N - 1, nx, nx, dtype=torch.float64)
        i = torch.arange(nu)
        A[..., i, i] = 1.0
        A[..., i, nu + i] = m["h"]
        A[..., nu + i, nu + i] = 1.0 - m["h"] * m["damping"]
        cs = m["coupling"] * torch.cos(q[..., 1:] - q[..., :-1])
        dg = -m["g"] * torch.cos(q)
        dg[..., :-1] -= cs
        dg[..., 1:] -= cs
        A[..., nu + i, i] = m["h"] * dg
        A[..., nu + i[:-1], i[1:]] = m["h"] * cs
        A[..., nu + i[1:], i[:-1]] = m["h"] * cs
        Bm = torch.zeros(B, N - 1, nx, nu, dtype=torch.float64)
        Bm[..., nu + i, i] = m["h"]
        p = dict(Q=Q.reshape(-1, nx, nx), R=R.reshape(-1, nu, nu), A=A.reshape(-1, nx, nx), B=Bm.reshape(-1, nx, nu),
                 q=_mv(Q, X - xr).reshape(-1, nx), r=_mv(R, U).reshape(-1, nu), x0=xi - X[:, 0],
                 e=(X[:, 1:] - _step64(m, X[:, :-1], U)).reshape(-1, nx))
        lam, dx, du = _solve64(_padded(p, [N] * B))
        du = du[:, :-1]
        mu = 1.0 + lam.abs().amax((1, 2))
        phi = torch.stack([cost(X + a * dx, U + a * du) + mu * viol(X + a * dx, U + a * du) for a in (2.0 ** -j for j in range(9))], 1)
        j = phi.argmin(1)
        a = (2.0 ** -j.double())[:, None, None]
        X, U = X + a * dx, U + a * du
    return dict(X=X.reshape(-1, nx), U=U.reshape(-1, nu), lam=lam.reshape(-1, nx), choice=None, status=None)


def exact(case, seed):
    kind = case["kind"]
    if kind == "control":
        return _control64(case, _trajectory(case, seed))
    p, Ns = _problem(case, seed), _horizons(case)
    d = _padded(p, Ns)
    if kind == "schur":
        return _schur64(d)
    lam, dx, du = _solve64(d)
    r = dict(lam=_knots(d, lam), dx=_knots(d, dx), du=_ctrls(d, du), status=None)
    if kind in ("train", "layer"):
        g = _grad64(d, lam, dx, du)
        r["grad"] = g if kind == "train" else {"d" + k: g["d" + k] for k in p}
    if kind == "train":
        r["status"] = [None, None]
    if kind == "layer":
        del r["status"]
    return r
