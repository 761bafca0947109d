"""Reduced mode and sEnKF for N > 128 over more rows than Q holds at a time (2^16):
a second panel of one row, of a part of its chunks, and a third panel; against a
64-bit solve, with the bars of test_reduced_wide_gpu.py (FP64 1e-10 and 1e-12)."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from tests.gpu_util import dev_problem, rel, run, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,N,k", [(65536, 129, 1), (65537, 130, 2), (70001, 200, 1),
                                   (131105, 140, 1)])
def test_panels(lib, m, N, k):
    say(f"case: panels m={m} N={N} k={k}")
    p = W.random_problem(300, m, N, k, seed=m + N, tol=1e-12)
    got = run(lib, p, "fp64", reduced=True, tol=1e-12, maxit=1000)
    ref = O.enkf_reduced(p.Xf, p.idx, p.w, p.y, p.r, p.eps)
    assert got["status"] == 0 and rel(got["Xa"], ref["Xa"]) <= 1e-10
    xa = lib.senkf_analysis(**dev_problem(p, "fp64"), prec="fp64")["Xa"].cpu().numpy()
    assert rel(xa, O.senkf(p.Xf, p.idx, p.w, p.y, p.r, p.eps)) <= 1e-12


@pytest.mark.parametrize("row", [3, 65536 + 7])
def test_bad_index_in_either_panel(lib, row):
    p = W.random_problem(300, 65600, 130, 1, seed=9)
    p.idx[row, 0] = 300
    assert run(lib, p, "fp64", reduced=True, raise_on_error=False)["status"] == -2
    d = dev_problem(p, "fp32")
    assert lib.senkf_analysis(**d, prec="fp32", raise_on_error=False)["status"] == -2
