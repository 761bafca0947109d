"""The analyses, network steps and batches whose speed matters, as cases.

A case is a dict of plain values.  listed() gives the standing cases, draw()
one more of the same ranges, prepare() what a program holds before the call
(device inputs, a plan or a workspace), run() one pass through the binding's
entry points, work() the bytes and operations a pass cannot do without and
exact() the same outputs in 64-bit torch arithmetic.

Kinds of case:
  analysis  binding.Plan, Algorithm 1 (full CG solve, N right-hand sides)
  tridiag   binding.analysis with a tridiagonal R (r_factor)
  reduced   binding.Plan(reduced=True), Algorithm 2
  senkf     binding.Plan(senkf=True), Appendix A
  batched   binding.Batch, many filters in one call
  gradient  WarmStartNet.loss_grad, the warm-start network forward and back

Models: "l96" is a Lorenz-96 twin experiment (members around a spun-up
truth), "field" a periodic two-dimensional Gaussian random field observed
bilinearly at random positions.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2606_19224_amd import binding

DEV = "cuda:0"


def listed():
    return [
        # Lorenz-96 with 40 variables: the smallest filter, one call a cycle,
        # where launches and latency are all there is
        dict(name="l96_40_fp64", kind="analysis", model="l96", n=40, m=20, N=20, k=1, r=1.0,
             prec="fp64", tol=1e-10, precond="none", spread_steps=0),
        # the twin experiment of the default benchmark: one analysis of a cycle
        dict(name="l96_twin_fp32", kind="analysis", model="l96", n=4096, m=2048, N=64, k=1, r=0.5,
             prec="fp32", tol=1e-6, precond="none", spread_steps=5),
        # double precision (the binding's default) at an ensemble of 100 and
        # sizes that fit no tile: random two-point observations, uneven R
        dict(name="ragged_fp64", kind="analysis", model="l96", n=8191, m=4093, N=100, k=2, r=0.0,
             prec="fp64", tol=1e-10, precond="none", spread_steps=5),
        # the two-dimensional field of the benchmark, in single precision ...
        dict(name="field_fp32", kind="analysis", model="field", ny=256, nx=256, m=16384, N=128,
             prec="fp32", tol=1e-6, precond="none"),
        # ... and in the BF16 mode with diag(R) preconditioning
        dict(name="field_mixed_pcg", kind="analysis", model="field", ny=256, nx=256, m=16384,
             N=128, prec="mixed", tol=1e-6, precond="diag_r"),
        # Example 2: every variable observed, tridiagonal R, 100 members
        dict(name="tridiag_fp32", kind="tridiag", model="l96", n=4096, m=4096, N=100, k=1,
             prec="fp32", tol=1e-6, spread_steps=0),
        # Algorithm 2 on the twin experiment: a few short launches
        dict(name="reduced_twin_fp32", kind="reduced", model="l96", n=4096, m=2048, N=64, k=1,
             r=0.5, prec="fp32", tol=1e-6, spread_steps=5),
        # Algorithm 2 in double precision on 10^5 observed variables and 100
        # members, a size of the paper's Table 5: streaming X_f and its product
        dict(name="reduced_wide_state_fp64", kind="reduced", model="l96", n=100000, m=100000,
             N=100, k=1, r=1.0, prec="fp64", tol=1e-10, spread_steps=0),
        # Algorithm 2 with more than 128 members
        dict(name="reduced_200_members_fp32", kind="reduced", model="l96", n=20011, m=5003, N=200,
             k=2, r=0.0, prec="fp32", tol=1e-6, spread_steps=5),
        # the comparison form on the field: one pass, no solve
        dict(name="senkf_field_fp32", kind="senkf", model="field", ny=256, nx=256, m=16384, N=128,
             prec="fp32"),
        # many uneven filters in one call
        dict(name="batched_64_fp32", kind="batched", count=64, n_lo=1024, n_hi=32768,
             sizes=7, prec="fp32", tol=1e-6),
        # one minibatch of the warm start's training: loss and gradient
        dict(name="train_64_pairs", kind="gradient", batch=64, m=2048),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["analysis", "analysis", "analysis", "tridiag", "reduced", "reduced",
                       "senkf", "batched", "gradient"])
    if kind == "gradient":
        return dict(kind=kind, batch=_log_int(rng, 4, 64), m=_log_int(rng, 40, 2048))
    if kind == "batched":
        return dict(kind=kind, count=_log_int(rng, 8, 64), n_lo=1024,
                    n_hi=_log_int(rng, 2048, 32768), sizes=rng.randrange(1 << 20), prec="fp32",
                    tol=1e-6)
    prec = rng.choice(["fp32", "fp64"])
    if kind == "senkf" or (kind == "analysis" and rng.random() < 0.4):
        ny, nx = rng.randrange(48, 257), rng.randrange(48, 257)
        case = dict(kind=kind, model="field", ny=ny, nx=nx, m=ny * nx // rng.choice([4, 5, 8]),
                    N=rng.randrange(24, 129), prec="fp32")
        if kind == "analysis":
            case["prec"] = rng.choice(["fp32", "mixed"])
            case["precond"] = rng.choice(["none", "diag_r"])
            case["tol"] = 1e-6
        return case
    tol = 1e-10 if prec == "fp64" else 1e-6
    if kind == "tridiag":
        n = _log_int(rng, 256, 4096)
        return dict(kind=kind, model="l96", n=n, m=n, N=rng.randrange(20, 101), k=1, prec=prec,
                    tol=tol, spread_steps=0)
    steps = rng.choice([0, 5])
    r = rng.choice([0.0, 0.5, 1.0])
    if kind == "reduced":
        N = rng.randrange(16, 201)
        n = _log_int(rng, 1000, 20011 if N > 100 else 100000)
        m = min(n // rng.choice([1, 2, 4]), 5003 if N > 100 else 100000)
        return dict(kind=kind, model="l96", n=n, m=m, N=N, k=1 if m == n else rng.choice([1, 2]),
                    r=r, prec=prec, tol=tol, spread_steps=steps)
    n = _log_int(rng, 40, 8191)
    return dict(kind=kind, model="l96", n=n, m=n // 2, N=_log_int(rng, 8, 100),
                k=rng.choice([1, 1, 2]), r=r, prec=prec, tol=tol,
                precond=rng.choice(["none", "none", "diag_r"]), spread_steps=steps)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 17)


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float64)


def _uniform(g, lo, hi, *shape):
    return lo + (hi - lo) * torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64)


def _l96_steps(x, steps, dt=0.05, forcing=8.0):
    def f(v):
        return (torch.roll(v, -1, 0) - torch.roll(v, 2, 0)) * torch.roll(v, 1, 0) - v + forcing
    for _ in range(steps):
        a = f(x)
        b = f(x + 0.5 * dt * a)
        c = f(x + 0.5 * dt * b)
        d = f(x + dt * c)
        x = x + (dt / 6.0) * (a + 2 * b + 2 * c + d)
    return x


def _observe(Xf, idx, w):
    out = torch.zeros(idx.shape[0], *Xf.shape[1:], dtype=Xf.dtype, device=Xf.device)
    for t in range(idx.shape[1]):
        wt = w[:, t] if Xf.dim() == 1 else w[:, t:t + 1]
        out += wt * Xf[idx[:, t].long()]
    return out


def _l96_problem(case, g):
    n, m, N, k = case["n"], case["m"], case["N"], case["k"]
    truth = _l96_steps(_normal(g, n), 200)
    X = truth[:, None] + _normal(g, n, N)
    if case["spread_steps"]:
        X = _l96_steps(X, case["spread_steps"])
        truth = _l96_steps(truth, case["spread_steps"])
    if k == 1 and m == n:          # every variable
        idx = torch.arange(n, device=DEV)[:, None]
    elif k == 1 and m == n // 2:   # every second variable
        idx = torch.arange(0, 2 * m, 2, device=DEV)[:, None]
    else:                          # random positions
        idx = torch.randint(0, n, (m, k), generator=g, device=DEV)
    w = torch.ones(m, k, device=DEV, dtype=torch.float64) if k == 1 else _uniform(g, 0.1, 1, m, k)
    r = case.get("r", 0.0)
    rv = torch.full((m,), r, device=DEV, dtype=torch.float64) if r else _uniform(g, 0.5, 2, m)
    return truth, X, idx, w, rv


def _field_problem(case, g):
    ny, nx, m, N = case["ny"], case["nx"], case["m"], case["N"]
    iy, ix = torch.arange(ny, device=DEV), torch.arange(nx, device=DEV)
    dy, dx = torch.minimum(iy, ny - iy).double(), torch.minimum(ix, nx - ix).double()
    cov = torch.exp(-(dy[:, None] ** 2 + dx[None, :] ** 2) / 128.0)  # length scale 8 cells
    amp = torch.fft.fft2(cov).real.clamp_min(0.0).sqrt()
    white = _normal(g, N + 1, ny, nx)
    f = torch.fft.ifft2(amp * torch.fft.fft2(white)).real.reshape(N + 1, ny * nx)
    px, py = _uniform(g, 0, nx, m), _uniform(g, 0, ny, m)
    x0, y0 = px.floor().long() % nx, py.floor().long() % ny
    fx, fy = px - px.floor(), py - py.floor()
    x1, y1 = (x0 + 1) % nx, (y0 + 1) % ny
    idx = torch.stack([y0 * nx + x0, y0 * nx + x1, y1 * nx + x0, y1 * nx + x1], 1)
    w = torch.stack([(1 - fx) * (1 - fy), fx * (1 - fy), (1 - fx) * fy, fx * fy], 1)
    return f[0].clone(), f[1:].t().contiguous(), idx, w, _uniform(g, 0.5, 2, m)


def _problem(case, seed):
    """Device inputs of one analysis, in the case's value type."""
    g = _generator(seed)
    dt = torch.float64 if case["prec"] == "fp64" else torch.float32
    truth, X, idx, w, r = (_field_problem if case["model"] == "field" else _l96_problem)(case, g)
    m, N = idx.shape[0], X.shape[1]
    p = {}
    if case["kind"] == "tridiag":
        # the paper's Example 2: sigma^2 on the diagonal, 0.2 sigma^2 beside it;
        # the noise is a moving average with that covariance
        s, rho = 0.3, 0.2
        a = 0.5 * (math.sqrt(1 + 2 * rho) + math.sqrt(1 - 2 * rho))
        b = 0.5 * (math.sqrt(1 + 2 * rho) - math.sqrt(1 - 2 * rho))
        u = _normal(g, m + 1, N + 1)
        noise = s * (a * u[:-1] + b * u[1:])
        r = torch.full((m,), s * s, device=DEV, dtype=torch.float64)
        p["r_off"] = torch.full((m - 1,), s * s * rho, device=DEV, dtype=dt)
    else:
        noise = r.sqrt()[:, None] * _normal(g, m, N + 1)
    y = _observe(truth, idx, w) + noise[:, 0]
    p.update(Xf=X.to(dt).contiguous(), idx=idx.to(torch.int32).contiguous(),
             w=w.to(dt).contiguous(), y=y.to(dt), r=r.to(dt),
             eps=noise[:, 1:].to(dt).contiguous())
    return p


def _batch_problems(case, seed):
    """Uneven Lorenz-96 filters: windows of one spun-up state, a quarter of
    the variables observed at random, R = I."""
    g = _generator(seed)
    base = _l96_steps(_normal(g, 32768), 200)
    rng = np.random.default_rng(case["sizes"])
    out = []
    for _ in range(case["count"]):
        n = 4 * int(rng.integers(case["n_lo"] // 4, case["n_hi"] // 4 + 1))
        m, N = n // 4, int(rng.choice([16, 32, 64]))
        off = int(rng.integers(0, 32768))
        truth = torch.roll(base, -off)[:n]
        X = truth[:, None] + _normal(g, n, N)
        idx = torch.randperm(n, generator=g, device=DEV)[:m].sort().values[:, None]
        e = _normal(g, m, N + 1)
        out.append(dict(Xf=X.float(), idx=idx.to(torch.int32), eps=e[:, 1:].float().contiguous(),
                        w=torch.ones(m, 1, device=DEV), y=(truth[idx[:, 0]] + e[:, 0]).float(),
                        r=torch.ones(m, device=DEV)))
    return out


def _pairs(case, seed):
    """Training pairs: normalised innovations, ensemble variance, R, and a
    target near the diagonal solution."""
    g = _generator(seed)
    B, m = case["batch"], case["m"]
    feat = torch.zeros(B, m, 4, device=DEV, dtype=torch.float64)
    feat[:, :, 0] = _normal(g, B, m)
    feat[:, :, 1] = _uniform(g, 0.5, 1.5, m)
    feat[:, :, 2] = 0.5
    target = feat[:, :, 0] / (feat[:, :, 1] + feat[:, :, 2])
    target = target + 0.2 * torch.roll(target, 1, 1) + 0.1 * _normal(g, B, m)
    return feat.float(), target.float()


# ---------------------------------------------------------------------------
# the calls
# ---------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    if kind == "gradient":
        feat, target = _pairs(case, seed)
        return dict(kind=kind, net=binding.WarmStartNet(seed=seed, device=DEV), feat=feat,
                    target=target)
    if kind == "batched":
        return dict(kind=kind, tol=case["tol"],
                    batch=binding.Batch(_batch_problems(case, seed), prec=case["prec"],
                                        tiles="auto"))
    p = _problem(case, seed)
    n, N = p["Xf"].shape
    m, k = p["idx"].shape
    state = dict(kind=kind, out=torch.empty_like(p["Xf"]))
    if kind == "tridiag":
        state["factor"] = binding.tridiag_cholesky(p["r"], p.pop("r_off"), prec=case["prec"])
        state["tol"], state["prec"] = case["tol"], case["prec"]
        state["workspace"] = torch.empty(
            binding.workspace_bytes(n, m, N, k, case["prec"], tridiag=True), dtype=torch.uint8,
            device=DEV)
    else:
        precond = case.get("precond", "none")
        state["plan"] = binding.Plan(n, m, N, k, prec=case["prec"], reduced=kind == "reduced",
                                     senkf=kind == "senkf", tol=case.get("tol", 1e-6),
                                     maxit=2000, device=DEV,
                                     precond=None if precond == "none" else precond)
    state["inputs"] = p
    return state


def run(state):
    kind = state["kind"]
    if kind == "gradient":
        loss, grad = state["net"].loss_grad(state["feat"], state["target"])
        return {"loss": loss, "grad": grad}
    if kind == "batched":
        state["batch"].run(tol=state["tol"], maxit=1000)
        return list(state["batch"].outs)
    p = state["inputs"]
    if kind == "tridiag":
        binding.analysis(**p, tol=state["tol"], maxit=2000, prec=state["prec"], stats=False,
                         out=state["out"], workspace=state["workspace"],
                         r_factor=state["factor"])
    else:
        state["plan"](p["Xf"], p["idx"], p["w"], p["y"], p["r"], p["eps"], state["out"])
    return state["out"]


# ---------------------------------------------------------------------------
# what a pass cannot do without, and its exact result
# ---------------------------------------------------------------------------
# CG steps an analysis takes at its tolerance: a property of the system, not of
# the code that solves it
_STEPS = {("l96", 1e-6): 17, ("l96", 1e-10): 40, ("field", "none"): 110, ("field", "diag_r"): 42}


def _analysis_work(n, m, N, k, b, steps):
    """Inputs once, X_a once; two products with S a step, S^T Z and the update."""
    read = n * N * b + m * k * (4 + b) + 2 * m * b + m * N * b
    return read + n * N * b, 4 * m * N * N * steps + 2 * m * N * N + 2 * n * N * N


def work(case):
    kind = case["kind"]
    if kind == "gradient":
        # forward, backward over the data (not into the features) and over the
        # weights; features, target, parameters and gradient once
        macs = 5 * (3 * 64 + 64 * 64 + 64 * 64 + 64)
        fl = 2 * case["batch"] * case["m"] * (3 * macs - 5 * 3 * 64)
        return {"bytes": 20 * case["batch"] * case["m"] + 8 * (macs + 193), "flops": fl}
    if kind == "batched":
        rng = np.random.default_rng(case["sizes"])
        tot = [0, 0]
        for _ in range(case["count"]):
            n = 4 * int(rng.integers(case["n_lo"] // 4, case["n_hi"] // 4 + 1))
            N = int(rng.choice([16, 32, 64]))
            rng.integers(0, 32768)
            by, fl = _analysis_work(n, n // 4, N, 1, 4, 11)
            tot = [tot[0] + by, tot[1] + fl]
        return {"bytes": tot[0], "flops": tot[1]}
    field = case["model"] == "field"
    n = case["ny"] * case["nx"] if field else case["n"]
    k = 4 if field else case["k"]
    b = 8 if case["prec"] == "fp64" else 4
    m, N = case["m"], case["N"]
    if kind == "senkf":
        by, fl = _analysis_work(n, m, N, k, b, 0)
    elif kind == "reduced":
        # the symmetric half of P^T P in place of the CG's products with S
        by, fl = _analysis_work(n, m, N, k, b, 0)
        fl += m * N * N + 2 * N * N * N * 20
    else:
        steps = _STEPS[("field", case["precond"]) if field else ("l96", case["tol"])]
        by, fl = _analysis_work(n, m, N, k, b, steps)
    return {"bytes": by, "flops": fl}


def _exact_analysis(p, kind):
    q = {key: v.double() if v.is_floating_point() else v for key, v in p.items()}
    Xf, idx, w, r = q["Xf"], q["idx"], q["w"], q["r"]
    N = Xf.shape[1]
    HX = _observe(Xf, idx, w)
    S = HX - HX.mean(1, keepdim=True)
    D = q["y"][:, None] + q["eps"] - HX
    if kind == "senkf":
        return Xf + Xf @ (S.t() @ (D / ((S * S).sum(1) + (N - 1) * r)[:, None]))
    if kind == "tridiag":
        R = torch.diag(r) + torch.diag(q["r_off"], 1) + torch.diag(q["r_off"], -1)
        RS = torch.linalg.solve(R, S)
    else:
        RS = S / r[:, None]
    G = RS.t() @ S
    G.diagonal().add_(N - 1.0)
    W = torch.linalg.solve(G, RS.t() @ D)
    return Xf + (Xf - Xf.mean(1, keepdim=True)) @ W


def _exact_gradient(case, seed):
    feat, target = (v.double() for v in _pairs(case, seed))
    vec = torch.as_tensor(binding.wsnet_init_params(seed), device=DEV).double().requires_grad_(True)
    x, at = feat[:, :, :3], 0
    for layer, (cin, cout) in enumerate(((3, 64), (64, 64), (64, 64), (64, 1))):
        W = vec[at:at + cout * cin * 5].reshape(cout, cin, 5)
        bias = vec[at + cout * cin * 5:at + cout * (cin * 5 + 1)]
        at += cout * (cin * 5 + 1)
        x = sum(torch.roll(x, 2 - t, 1) @ W[:, :, t].t() for t in range(5)) + bias
        if layer < 3:
            x = torch.relu(x)
    loss = ((x[:, :, 0] - target) ** 2).mean()
    (grad,) = torch.autograd.grad(loss, vec)
    return {"loss": loss.detach().reshape(1), "grad": grad}


def exact(case, seed):
    kind = case["kind"]
    if kind == "gradient":
        return _exact_gradient(case, seed)
    if kind == "batched":
        return [_exact_analysis(p, kind) for p in _batch_problems(case, seed)]
    return _exact_analysis(_problem(case, seed), kind)
