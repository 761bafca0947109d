"""FP32 batches: which of the two solvers runs (one member a workgroup, or groups of
four where those fill the GPU), and parity of both, captured or not, at the edges of
the group solver's row tiles (64), waves (8 tiles), column paddings (16, 32, 64) and of
the last group of members.  FP32 bar 1e-4."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from tests.gpu_util import dev_problem, rel, rounded, say

pytestmark = pytest.mark.gpu

SIZES = [(30, 1, 2, 1), (80, 63, 3, 2), (90, 64, 5, 1), (90, 65, 16, 4), (600, 511, 17, 1),
         (600, 512, 32, 2), (700, 513, 33, 3), (1217, 400, 44, 2), (1500, 1089, 47, 1),
         (4000, 2111, 63, 2), (4000, 3000, 64, 1)]
FEW = [(80, 63, 3, 2), (90, 65, 16, 4), (600, 511, 17, 1), (600, 512, 32, 2), (600, 513, 31, 1),
       (4000, 2111, 5, 3), (900, 700, 9, 1)]   # at most 32 members on an XCD


def _args(p):
    return {k: v for k, v in dev_problem(p, "fp32").items()}


def _batch(lib, probs, copies, **kw):
    return lib.Batch([_args(p) for _ in range(copies) for p in probs], prec="fp32", **kw)


@pytest.mark.parametrize("m,N,count,members", [
    (256, 16, 1, 4), (257, 16, 1, 1), (500, 16, 16, 1), (2000, 16, 17, 4), (2000, 32, 8, 1),
    (2000, 32, 9, 4), (2000, 33, 1, 4), (20, 40, 1, 4), (2000, 64, 4, 4), (2000, 8, 32, 1)])
def test_choice(lib, m, N, count, members):
    p = _args(W.random_problem(2 * m, m, N, 1, seed=m + N))
    assert lib.Batch([p] * count, prec="fp32").plan.members == members
    d = {k: v.double() if v.is_floating_point() else v for k, v in p.items()}
    assert lib.Batch([d], prec="fp64").plan.members == 1


@pytest.mark.parametrize("precond", [None, "diag_r"])
@pytest.mark.parametrize("sizes,copies,members", [(FEW, 1, 1), (SIZES, 1, 4), (SIZES, 3, 4)])
def test_parity_of_both(lib, sizes, copies, members, precond):
    import torch
    probs = [rounded(W.random_problem(n, m, N, k, seed=800 + i, tol=1e-6))
             for i, (n, m, N, k) in enumerate(sizes)]
    say(f"case: batched choice copies={copies} precond={precond}")
    b = _batch(lib, probs, copies, precond=precond)
    assert b.plan.members == members
    status, stats = b.run(tol=1e-6, maxit=1000, stats=True)
    torch.cuda.synchronize()
    assert status == 0 and all(st["n_converged"] == p.N for p, st in zip(probs * copies, stats))
    first = [o.clone() for o in b.outs]
    for i, p in enumerate(probs):
        ref = O.enkf_analysis(p.Xf, p.idx, p.w, p.y, p.r, p.eps, solver="cg_free", tol=1e-6,
                              maxit=1000)["Xa"]
        for c in range(copies):   # every copy is the same problem
            assert torch.equal(first[i], first[i + c * len(probs)])
        assert rel(first[i].cpu().numpy(), ref) <= 1e-4, p.name
    b.run(tol=0.0, maxit=2)
    torch.cuda.synchronize()
    for p, out, it in zip(probs, b.outs, b.iters):
        if p.m >= 20:   # (two steps may pass exact termination)
            assert np.all(it.cpu().numpy() == 2)
    # captured, replayed on other values, against an uncaptured run
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        b.run(tol=1e-6, maxit=1000)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        b.run(tol=1e-6, maxit=1000)
    for scale in (1.0, 0.5, 1.0):
        for q in b.problems:
            q["y"].mul_(scale)
        g.replay()
        torch.cuda.synchronize()
        got = [o.clone() for o in b.outs]
        b.run(tol=1e-6, maxit=1000)
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(got, b.outs))


def test_bad_index_in_either(lib):
    p = W.random_problem(300, 400, 16, 1, seed=3)
    q = W.random_problem(300, 400, 16, 1, seed=4)
    q.idx[399, 0] = 300
    for count, members in ((1, 1), (80, 4)):
        b = lib.Batch([_args(p)] * count + [_args(q)], prec="fp32")
        assert b.plan.members == members
        with pytest.raises(lib.CGDError):
            b.run(stats=True)


def test_many_rows_in_groups(lib):
    """One filter of 2 * 10^5 rows in groups of four: 391 rows a lane in its FP32 sums."""
    p = rounded(W.random_problem(500, 200_000, 40, 1, seed=12, tol=1e-6))
    b = lib.Batch([_args(p)], prec="fp32", precond="diag_r")
    assert b.plan.members == 4
    status, stats = b.run(tol=1e-6, maxit=1000, stats=True)
    assert status == 0 and stats[0]["n_converged"] == 40
    ref = O.enkf_reduced(p.Xf, p.idx, p.w, p.y, p.r, p.eps)["Xa"]   # the same analysis
    assert rel(b.outs[0].cpu().numpy(), ref) <= 1e-4
