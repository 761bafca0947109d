"""Reduced mode, sEnKF and full mode for N > 128 (padded to 64, on-chip N x N
CG to 256, the wide update) at the edges of their widths, against the oracle:
FP64 1e-10 (sEnKF 1e-12) and FP32 1e-4 on X_a, the bars of the other modes.
The products are FP64 in both precisions."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from tests.gpu_util import assert_iters_close, dev_problem, rel, rounded, run, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,N,k", [(33, 5, 129, 1), (500, 40, 191, 2), (310, 257, 192, 1),
                                     (400, 300, 193, 3), (1000, 700, 256, 2), (200, 321, 257, 1),
                                     (90, 64, 520, 2)])
def test_reduced_and_senkf_widths(lib, n, m, N, k):
    import torch
    say(f"case: reduced wide n={n} m={m} N={N} k={k}")
    p = W.random_problem(n, m, N, k, seed=n + N, tol=1e-12)
    got = run(lib, p, "fp64", reduced=True, tol=1e-12, maxit=1000, want_iters=True)
    ref = O.enkf_reduced(p.Xf, p.idx, p.w, p.y, p.r, p.eps, solver="cg", tol=1e-12, maxit=1000)
    assert rel(got["Xa"], ref["Xa"]) <= 1e-10
    assert_iters_close(got["iters"], ref["iters"])
    q = rounded(p)
    f32 = run(lib, p, "fp32", reduced=True, tol=1e-7)
    assert rel(f32["Xa"], O.enkf_reduced(q.Xf, q.idx, q.w, q.y, q.r, q.eps)["Xa"]) <= 1e-4
    d = dev_problem(p, "fp64")
    sen = lib.senkf_analysis(**d, prec="fp64")["Xa"]
    torch.cuda.synchronize()
    assert rel(sen.cpu().numpy(), O.senkf(p.Xf, p.idx, p.w, p.y, p.r, p.eps)) <= 1e-12
    # in place, and bitwise repeatable
    Xf = d["Xf"].clone()
    lib.senkf_analysis(**dict(d, Xf=Xf), prec="fp64", out=Xf)
    assert torch.equal(Xf, sen)


@pytest.mark.parametrize("prec,N", [("fp64", 65), ("fp64", 112), ("fp64", 128), ("fp64", 300),
                                    ("fp32", 144)])
def test_wide_update_in_full_mode(lib, prec, N):
    """Mode 0 of the wide update (centred rows): tol 1 keeps X_f exactly, a
    solve matches the oracle; n leaves a part tile."""
    say(f"case: wide update {prec} N={N}")
    p = W.random_problem(161, 90, N, 2, seed=N, tol=1e-12 if prec == "fp64" else 1e-7)
    got = run(lib, p, prec, tol=p.tol, maxit=2000)
    q = p if prec == "fp64" else rounded(p)
    ref = O.enkf_analysis(q.Xf, q.idx, q.w, q.y, q.r, q.eps)
    assert rel(got["Xa"], ref["Xa"]) <= (1e-10 if prec == "fp64" else 1e-4)
    same = run(lib, p, prec, tol=1.0)
    assert np.array_equal(same["Xa"], q.Xf)
