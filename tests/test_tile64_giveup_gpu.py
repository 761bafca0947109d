"""The FP64 row-block solver (64 < N <= 128) when a wait for another workgroup runs
out, forced by a limit of one tick (10 ns) that no exchange meets: every workgroup
returns, the call reports CGD_ERR_HIP, X_a and an in-place X_f stay as they were,
and the next call on the same workspace is right."""
import pytest

import workloads as W
from tests.gpu_util import dev_problem, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,N,precond", [(1800, 65, None), (2500, 100, "diag_r"), (4096, 128, None)])
def test_a_wait_that_runs_out_leaves_x_a_alone(lib, m, N, precond):
    import torch
    say(f"case: tile64 give-up m={m} N={N}")
    p = W.random_problem(2 * m, m, N, 1, seed=m + N, tol=1e-10)
    d = dev_problem(p, "fp64")
    kw = dict(tol=1e-10, maxit=1000, prec="fp64", precond=precond)
    assert lib.Plan(2 * m, m, N, 1, prec="fp64").solver_info()["solver"] == "k_cg_tile"
    ref = lib.analysis(**d, **kw)
    ws = ref["workspace"]
    sentinel = torch.full_like(ref["Xa"], 7.0)
    out = lib.analysis(**d, **kw, census_ticks=1, workspace=ws, raise_on_error=False,
                       out=sentinel.clone())
    torch.cuda.synchronize()
    assert out["status"] == -6 and torch.equal(out["Xa"], sentinel)
    Xf = d["Xf"].clone()
    out = lib.analysis(**dict(d, Xf=Xf), **kw, census_ticks=1, workspace=ws, stats=False, out=Xf)
    torch.cuda.synchronize()
    assert torch.equal(Xf, d["Xf"])
    again = lib.analysis(**d, **kw, workspace=ws)
    torch.cuda.synchronize()
    assert again["status"] == 0 and torch.equal(again["Xa"], ref["Xa"])
