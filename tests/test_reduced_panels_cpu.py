"""Workspace of the reduced mode and the sEnKF for N > 128: past 2^16 rows it does not
grow with m, and holds no more than 1024 N x 2N sums in double (and the N x N arrays)."""
import pytest

from paper_2606_19224_amd import binding


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("N", [129, 130, 192, 200, 256, 300, 512])
def test_workspace_stops_growing(prec, N):
    size = lambda m: binding.workspace_bytes(m, m, N, 1, prec, reduced=True)
    assert size(1_000_000) == size(4_000_000) == size(1 << 16)
    assert size(4_000_000) <= 1024 * 16 * N * N + 64 * N * N
