"""Reduced mode and sEnKF for 64 < N <= 128, or more than 8192 rows: the gather
and product launch at the edges of its member tiles (16), row chunks (32) and workgroups (256
chunks at once), against the oracle with the bars of test_reduced_gpu.py and
test_senkf_gpu.py (FP64 1e-10 and 1e-12, FP32 1e-4 and 1e-5)."""
import pytest
import torch

import oracle as O
import workloads as W
from tests.gpu_util import assert_iters_close, dev_problem, rel, rounded, run, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,N,k", [(40, 1, 65, 1), (50, 31, 80, 2), (60, 32, 81, 1),
                                     (70, 33, 96, 5), (90, 65, 97, 1), (100, 300, 112, 2),
                                     (120, 96, 113, 3), (200, 8192, 128, 1), (300, 8225, 100, 2),
                                     (150, 20000, 72, 1), (90, 8193, 9, 1), (90, 8300, 32, 2),
                                     (90, 16500, 47, 1), (90, 8192, 64, 1), (90, 8200, 64, 3)])
def test_chunk_and_tile_edges(lib, n, m, N, k):
    say(f"case: reduced stream n={n} m={m} N={N} k={k}")
    p = W.random_problem(n, m, N, k, seed=n + N, tol=1e-12)
    q = rounded(p)
    got = run(lib, p, "fp64", reduced=True, tol=1e-12, maxit=1000, want_iters=True)
    ref = O.enkf_reduced(p.Xf, p.idx, p.w, p.y, p.r, p.eps, solver="cg", tol=1e-12, maxit=1000)
    assert rel(got["Xa"], ref["Xa"]) <= 1e-10
    assert_iters_close(got["iters"], ref["iters"])
    f32 = run(lib, p, "fp32", reduced=True, tol=1e-7)
    assert rel(f32["Xa"], O.enkf_reduced(q.Xf, q.idx, q.w, q.y, q.r, q.eps)["Xa"]) <= 1e-4
    for prec, src, bar in (("fp64", p, 1e-12), ("fp32", q, 1e-5)):
        d = dev_problem(p, prec)
        a = lib.senkf_analysis(**d, prec=prec)["Xa"].clone()
        b = lib.senkf_analysis(**d, prec=prec)["Xa"]
        torch.cuda.synchronize()
        assert torch.equal(a, b)
        assert rel(a.cpu().numpy(), O.senkf(src.Xf, src.idx, src.w, src.y, src.r, src.eps)) <= bar


def test_bad_index_is_reported(lib):
    p = W.random_problem(200, 9000, 90, 2, seed=5)
    p.idx[8999, 1] = 200
    assert run(lib, p, "fp64", reduced=True, raise_on_error=False)["status"] == -2
    d = dev_problem(p, "fp32")
    assert lib.senkf_analysis(**d, prec="fp32", raise_on_error=False)["status"] == -2
