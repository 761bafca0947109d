"""Streamed reduced mode and sEnKF on either side of their lines: four workgroups a
chunk of 32 rows up to 64 chunks (N > 64), one past that, and for N <= 64 a part per
chunk up to 256 chunks, in FP32 reduced mode 384.  Bars of test_reduced_gpu.py and
test_senkf_gpu.py (FP64 1e-10 and 1e-12, FP32 1e-4 and 1e-5)."""
import pytest

import oracle as O
import workloads as W
from tests.gpu_util import dev_problem, rel, rounded, run, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,N,k", [(70, 1, 128, 1), (90, 40, 65, 3), (300, 2016, 96, 1),
                                     (300, 2048, 128, 2), (300, 2049, 128, 1), (300, 2049, 70, 6),
                                     (90, 8225, 20, 1), (90, 12288, 64, 1), (90, 12289, 64, 2),
                                     (90, 12300, 33, 1)])
def test_both_sides(lib, n, m, N, k):
    say(f"case: reduced split n={n} m={m} N={N} k={k}")
    p = W.random_problem(n, m, N, k, seed=n + m + N, tol=1e-12)
    q = rounded(p)
    got = run(lib, p, "fp64", reduced=True, tol=1e-12, maxit=1000)
    assert rel(got["Xa"], O.enkf_reduced(p.Xf, p.idx, p.w, p.y, p.r, p.eps)["Xa"]) <= 1e-10
    f32 = run(lib, p, "fp32", reduced=True, tol=1e-7)
    assert rel(f32["Xa"], O.enkf_reduced(q.Xf, q.idx, q.w, q.y, q.r, q.eps)["Xa"]) <= 1e-4
    for prec, src, bar in (("fp64", p, 1e-12), ("fp32", q, 1e-5)):
        xa = lib.senkf_analysis(**dev_problem(p, prec), prec=prec)["Xa"].cpu().numpy()
        assert rel(xa, O.senkf(src.Xf, src.idx, src.w, src.y, src.r, src.eps)) <= bar


@pytest.mark.parametrize("m", [33, 2040])
def test_bad_index_with_four_workgroups_a_chunk(lib, m):
    p = W.random_problem(200, m, 90, 2, seed=6)
    p.idx[m - 1, 1] = 200
    assert run(lib, p, "fp64", reduced=True, raise_on_error=False)["status"] == -2
    assert lib.senkf_analysis(**dev_problem(p, "fp32"), prec="fp32",
                              raise_on_error=False)["status"] == -2
