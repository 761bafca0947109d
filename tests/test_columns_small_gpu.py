"""Analyses with few observation rows (up to 64 rows, or 128 with up to 32
members in FP64 and 64 in FP32), whose members are solved by one wave each:
parity with the oracle at the edges of the rows per lane (64, 128) and of the
column paddings (16, 32, 64), with preconditioning, fixed iterations, a zero
iteration cap and in place.  Bars 1e-10 (FP64) and
1e-4 (FP32)."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from tests.gpu_util import assert_iters_close, dev_problem, rel, rounded, run, say

pytestmark = pytest.mark.gpu

SIZES = [(20, 1, 2, 1), (40, 20, 20, 1), (70, 63, 16, 4), (100, 64, 17, 1), (100, 64, 64, 2),
         (90, 65, 32, 1), (150, 127, 15, 2), (200, 128, 32, 1), (200, 128, 33, 1),
         (130, 65, 63, 2), (300, 129, 16, 1), (9, 7, 48, 1)]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n,m,N,k", SIZES)
def test_parity(lib, n, m, N, k, prec):
    import torch
    say(f"case: {prec} few rows n={n} m={m} N={N} k={k}")
    bar, tol = (1e-10, 1e-12) if prec == "fp64" else (1e-4, 1e-6)
    p = W.random_problem(n, m, N, k, seed=n + m + N, tol=tol)
    if prec == "fp32":
        p = rounded(p)
    got = run(lib, p, prec, want_z=True, want_iters=True, want_relres=True)
    ref = O.enkf_analysis(p.Xf, p.idx, p.w, p.y, p.r, p.eps, solver="cg_free", tol=tol,
                          maxit=p.maxit)
    assert got["status"] == 0
    assert rel(got["Xa"], ref["Xa"]) <= bar
    assert got["relres"].max() <= (1e-10 if prec == "fp64" else 1e-5)
    if prec == "fp64":   # (FP32 stops within tol kappa of the solution, not within the bar)
        assert rel(got["Z"], ref["Z"]) <= bar
        assert_iters_close(got["iters"], ref["iters"])
    fixed = run(lib, p, prec, tol=0.0, maxit=3, want_z=True, want_iters=True)
    want = O.enkf_analysis(p.Xf, p.idx, p.w, p.y, p.r, p.eps, solver="cg_free", tol=0.0, maxit=3)
    if min(m, N) >= 15:   # (with fewer distinct eigenvalues three steps may pass termination)
        assert np.all(fixed["iters"] == 3) and rel(fixed["Z"], want["Z"]) <= bar
    none = run(lib, p, prec, tol=0.0, maxit=0, want_z=True, want_iters=True)
    assert np.all(none["iters"] == 0) and np.all(none["Z"] == 0) and rel(none["Xa"], p.Xf) <= 1e-15
    chol = O.enkf_analysis(p.Xf, p.idx, p.w, p.y, p.r, p.eps)
    pre = run(lib, p, prec, precond="diag_r", want_z=True)
    assert rel(pre["Xa"], chol["Xa"]) <= bar
    if prec == "fp64":
        assert rel(pre["Z"], chol["Z"]) <= bar
    a = dev_problem(p, prec)
    first = lib.analysis(**a, tol=tol, maxit=p.maxit, prec=prec)["Xa"].clone()
    inplace = lib.analysis(**a, tol=tol, maxit=p.maxit, prec=prec, out=a["Xf"], stats=False)
    torch.cuda.synchronize()
    assert torch.equal(first, inplace["Xa"])   # repeatable, and X_a may alias X_f


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_launch_modes_capture_and_bad_index(lib, prec):
    import torch
    bar = 1e-10 if prec == "fp64" else 1e-4
    tol = 1e-12 if prec == "fp64" else 1e-6
    p = W.random_problem(60, 30, 20, 2, seed=5, tol=tol)
    q = W.random_problem(60, 30, 20, 2, seed=6, tol=tol)
    want = [O.enkf_analysis(x.Xf, x.idx, x.w, x.y, x.r, x.eps)["Xa"] for x in (p, q)]
    assert rel(run(lib, p, prec, cooperative=True)["Xa"], want[0]) <= bar
    assert rel(run(lib, p, prec, solver=3)["Xa"], want[0]) <= bar
    # captured once, replayed on changed inputs with eager work in between
    a, b = dev_problem(p, prec), dev_problem(q, prec)
    plan = lib.Plan(60, 30, 20, 2, prec=prec, tol=tol, maxit=1000)
    out = torch.empty_like(a["Xf"])
    plan(a["Xf"], a["idx"], a["w"], a["y"], a["r"], a["eps"], out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan(a["Xf"], a["idx"], a["w"], a["y"], a["r"], a["eps"], out)
    first = {k: v.clone() for k, v in a.items() if v is not None}
    for which in (0, 1, 0, 1):
        for k, v in (first, b)[which].items():
            if v is not None:
                a[k].copy_(v)
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert rel(out.double().cpu().numpy(), want[which]) <= bar
    p.idx[7, 0] = 60
    assert run(lib, p, prec, raise_on_error=False)["status"] == -2
