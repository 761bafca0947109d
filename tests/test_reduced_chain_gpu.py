"""Reduced mode and sEnKF in FP32 over many observation rows: the N x 2N sums
must not lose accuracy as m grows.

Every row is the same observation, so all rows round alike and the rounding of
an FP32 chain adds up instead of averaging out; the product is m times one outer
product, known exactly.  With scale = m |p|^2 the perturbation of G = I + P^T P
passes to W undamped off the observed direction, so the bar of the reduced mode
is scale (100) times the relative error of the longest FP32 sum.  N <= 64, 32 rows:
two rounded operands and eight additions whose k-th sum is k/8 of the total, about 3
units of 2^-24 together, 2e-5.  N > 64, 512 rows: 128 such additions, in the last
half of which equal addends round alike, at most half a unit each of about three
quarters of the total, a third of that allowed for (20 units), 1.2e-4.  (Chains over
a workgroup's 4096 rows of this case gave 3e-4 to 7e-4.)  The sEnKF has no solve: W of order one, the same units and the FP32 update's
own, 2e-6."""
import numpy as np
import pytest
import torch

from tests.gpu_util import rel, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [16, 48, 64, 100])
def test_sums_over_a_million_equal_rows(lib, N):
    m, n, y = 1 << 20, 64, 0.7
    say(f"case: equal rows m={m} N={N}")
    X = np.random.default_rng(N).standard_normal((n, N)).astype(np.float32)
    h = X[5].astype(np.float64)
    s = h - h.mean()
    y = float(np.float32(y))

    def problem(scale):
        r = float(np.float32(m * (s @ s) / ((N - 1) * scale)))
        full = lambda v, *shape: torch.full(shape, v, dtype=torch.float32, device="cuda:0")
        d = dict(Xf=torch.as_tensor(X, device="cuda:0"), y=full(y, m), r=full(r, m), w=full(1.0, m, 1),
                 idx=torch.full((m, 1), 5, dtype=torch.int32, device="cuda:0"))
        return d, r

    d, r = problem(100.0)
    l2 = (N - 1) * r
    G = np.eye(N) + m * np.outer(s, s) / l2
    B = np.eye(N) + m * np.outer(s, np.full(N, y - h.mean())) / l2
    got = lib.analysis(**d, tol=1e-9, maxit=200, prec="fp32", reduced=True)["Xa"]
    assert rel(got.cpu().numpy(), X.astype(np.float64) @ np.linalg.solve(G, B)) <= (2e-5 if N <= 64 else 1.2e-4)

    d, r = problem(1.0)
    l2 = s @ s + (N - 1) * r
    W = m * np.outer(s, y - h) / l2
    got = lib.senkf_analysis(**d, prec="fp32")["Xa"]
    assert rel(got.cpu().numpy(), X.astype(np.float64) @ (np.eye(N) + W)) <= 2e-6
