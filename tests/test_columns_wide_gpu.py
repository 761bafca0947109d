"""FP64 analyses with 64 < N <= 128 (the row-block x member-group solver in
FP64, and the column solver with its own update launch for few rows and warm
starts): parity with the oracle's textbook CG at the edges of their row blocks
(128) and row steps (64), of the column solver's LDS vectors (about 3000
rows) and of N, with a warm start, preconditioning, fixed iterations and in
place.  FP64 bar 1e-10."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from tests.gpu_util import assert_iters_close, dev_problem, rel, run, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,N,k", [(50, 1, 65, 1), (80, 20, 128, 2), (200, 63, 96, 1),
                                     (200, 64, 100, 3), (300, 65, 66, 1), (900, 700, 127, 4),
                                     (700, 1799, 81, 1), (700, 1800, 128, 2), (1500, 3073, 100, 1),
                                     (900, 6528, 80, 1)])
def test_parity(lib, n, m, N, k):
    import torch
    say(f"case: fp64 columns n={n} m={m} N={N} k={k}")
    assert lib.Plan(n, m, N, k, prec="fp64").solver_info()["solver"] in ("k_cg_columns",
                                                                         "k_cg_tile")
    p = W.random_problem(n, m, N, k, seed=n + m, tol=1e-12)
    got = run(lib, p, "fp64", want_z=True, want_iters=True, want_relres=True)
    ref = O.enkf_analysis(p.Xf, p.idx, p.w, p.y, p.r, p.eps, solver="cg_free", tol=p.tol,
                          maxit=p.maxit)
    assert got["status"] == 0
    assert rel(got["Xa"], ref["Xa"]) <= 1e-10 and rel(got["Z"], ref["Z"]) <= 1e-10
    assert_iters_close(got["iters"], ref["iters"])
    assert got["relres"].max() <= 1e-10
    fixed = run(lib, p, "fp64", tol=0.0, maxit=4, want_z=True, want_iters=True)
    want = O.enkf_analysis(p.Xf, p.idx, p.w, p.y, p.r, p.eps, solver="cg_free", tol=0.0, maxit=4)
    if m >= 20:   # (with fewer rows four steps pass exact termination)
        assert np.all(fixed["iters"] == 4) and rel(fixed["Z"], want["Z"]) <= 1e-10
    a = dev_problem(p, "fp64")
    first = lib.analysis(**a, tol=p.tol, maxit=p.maxit, prec="fp64")["Xa"].clone()
    inplace = lib.analysis(**a, tol=p.tol, maxit=p.maxit, prec="fp64", out=a["Xf"], stats=False)
    torch.cuda.synchronize()
    assert torch.equal(first, inplace["Xa"])   # repeatable, and X_a may alias X_f


def test_warm_start_and_preconditioning(lib):
    import torch
    p = W.random_problem(1500, 1900, 90, 2, seed=77, tol=1e-12)
    chol = O.enkf_analysis(p.Xf, p.idx, p.w, p.y, p.r, p.eps)
    pre = run(lib, p, "fp64", precond="diag_r", want_z=True)
    assert rel(pre["Xa"], chol["Xa"]) <= 1e-10 and rel(pre["Z"], chol["Z"]) <= 1e-10
    plain = run(lib, p, "fp64", want_z=True, want_relres=True)
    assert rel(plain["Z"], chol["Z"]) <= 1e-10 and plain["relres"].max() <= 1e-10
    for scale in (1e-3, 30.0):   # a good start, and one that falls back to zero
        Z0 = chol["Z"] * (1 + scale * np.random.default_rng(3).standard_normal(chol["Z"].shape))
        z0 = torch.as_tensor(np.ascontiguousarray(Z0), device="cuda:0")
        got = run(lib, p, "fp64", z0=z0, fallback_on_stall=True, want_z=True)
        ref = O.enkf_analysis(p.Xf, p.idx, p.w, p.y, p.r, p.eps, solver="cg_free", tol=p.tol,
                              maxit=p.maxit, Z0=Z0, fallback_on_stall=True)
        assert got["stats"]["n_fallbacks"] == int(ref["fallbacks"].sum())
        assert rel(got["Z"], ref["Z"]) <= 1e-10


def test_bad_index_and_forced_solvers(lib):
    p = W.random_problem(200, 100, 80, 1, seed=78)
    p.idx[40, 0] = 200
    assert run(lib, p, "fp64", raise_on_error=False)["status"] == -2
    for solver, status in ((3, -7), (4, -7), (2, -7)):
        assert run(lib, p, "fp64", solver=solver, raise_on_error=False)["status"] == status
