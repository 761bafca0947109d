"""FP32 batched analyses, which solve four members of a filter per workgroup:
parity with the oracle at the edges of their row tiles (64), waves (8 tiles),
column paddings (16, 32, 64) and of the last group of members.  FP32 bar 1e-4.
And full-mode FP64 updates with 64 < N <= 128 from enough rows that their
weights stay in registers (32768).  FP64 bar 1e-10."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from tests.gpu_util import dev_problem, rel, rounded, run, say

pytestmark = pytest.mark.gpu

SIZES = [(30, 1, 2, 1), (80, 63, 3, 2), (90, 64, 5, 1), (90, 65, 16, 4), (600, 511, 17, 1),
         (600, 512, 32, 2), (700, 513, 33, 3), (1217, 400, 44, 2), (300, 90, 20, 1),
         (1500, 1089, 47, 1), (4000, 2111, 63, 2),
         (4000, 3000, 64, 1)]


def _args(p):
    d = dev_problem(p, "fp32")
    return {"Xf": d["Xf"], "idx": d["idx"], "w": d["w"], "y": d["y"], "r": d["r"], "eps": d["eps"]}


@pytest.mark.parametrize("precond", [None, "diag_r"])
@pytest.mark.parametrize("det", [False, True])
def test_groups_of_four(lib, det, precond):
    import torch
    probs = [rounded(W.random_problem(n, m, N, k, seed=700 + i, tol=1e-6, stochastic=not det))
             for i, (n, m, N, k) in enumerate(SIZES)]
    say(f"case: batched fp32 groups det={det} precond={precond}")
    b = lib.Batch([_args(p) for p in probs], prec="fp32", precond=precond)
    status, stats = b.run(tol=1e-6, maxit=1000, stats=True)
    torch.cuda.synchronize()
    assert status == 0
    first = [o.clone() for o in b.outs]
    for p, out, st in zip(probs, first, stats):
        ref = O.enkf_analysis(p.Xf, p.idx, p.w, p.y, p.r, p.eps, solver="cg_free", tol=1e-6,
                              maxit=1000)
        assert rel(out.cpu().numpy(), ref["Xa"]) <= 1e-4, p.name
        assert st["n_converged"] == p.N
    b.run(tol=1e-6, maxit=1000)
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(first, b.outs))
    for maxit in (0, 2):
        b.run(tol=0.0, maxit=maxit)
        torch.cuda.synchronize()
        for p, out, it in zip(probs, b.outs, b.iters):
            if p.m < 20:
                continue   # (two steps may pass exact termination)
            assert np.all(it.cpu().numpy() == maxit)
            if precond is None or maxit == 0:
                ref = O.enkf_analysis(p.Xf, p.idx, p.w, p.y, p.r, p.eps, solver="cg_free",
                                      tol=0.0, maxit=maxit)
                assert rel(out.cpu().numpy(), ref["Xa"]) <= 1e-4, p.name


@pytest.mark.parametrize("n,m,N", [(32768, 300, 65), (32769, 200, 100), (40003, 300, 128)])
def test_full_mode_update_fp64(lib, n, m, N):
    say(f"case: fp64 full-mode update n={n} m={m} N={N}")
    p = W.random_problem(n, m, N, 1, seed=n + N, tol=1e-12)
    got = run(lib, p, "fp64", want_z=True)
    ref = O.enkf_analysis(p.Xf, p.idx, p.w, p.y, p.r, p.eps, solver="cg_free", tol=1e-12, maxit=1000)
    assert got["status"] == 0
    assert rel(got["Xa"], ref["Xa"]) <= 1e-10 and rel(got["Z"], ref["Z"]) <= 1e-10
