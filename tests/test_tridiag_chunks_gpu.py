"""The whitening pass's chunked forward substitution (chunks of 32 rows; the
members kept in LDS up to N = 256) at the edges of its chunks, full and
reduced mode in FP64 against the oracle's direct solutions (1e-10, the FP64
bar of test_tridiag_gpu.py)."""
import pytest

import oracle as O
from tests.gpu_util import rel, say
from tests.test_tridiag_gpu import _run, _tri

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,N", [(1, 2), (2, 5), (31, 20), (32, 20), (33, 7), (65, 33),
                                 (545, 100), (70, 256), (70, 257)])
def test_chunk_edges(lib, m, N):
    p, ro = _tri(200, m, N, 2, seed=5300 + m + N)
    R = O.tridiag_R(p.r, ro)
    say(f"case: tridiagonal R chunk edges m={m} N={N}")
    ref = O.enkf_reduced_R(p.Xf, p.idx, p.w, p.y, R, p.eps)["Xa"]   # = Algorithm 1's X_a
    got = _run(lib, p, ro, tol=1e-13, maxit=1000, prec="fp64", reduced=True)
    assert rel(got["Xa"], ref) <= 1e-10
    if N <= 100:
        full = _run(lib, p, ro, tol=1e-12, maxit=2000, prec="fp64", want_z=True)
        assert rel(full["Xa"], ref) <= 1e-10
