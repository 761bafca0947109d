"""Which solver an FP64 analysis with 64 < N <= 128 runs: the row-block solver from 1800
rows while its workgroups fit the GPU, the column solver for fewer or more rows and
for warm starts, the streaming solver past the rows where that is the faster one."""
import pytest

import oracle as O
import workloads as W
from tests.gpu_util import dev_problem, rel, run, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,N,want", [(1, 65, "k_cg_columns"), (1799, 81, "k_cg_columns"),
                                      (1800, 128, "k_cg_tile"), (1800, 65, "k_cg_tile"),
                                      (3073, 100, "k_cg_tile"), (4096, 128, "k_cg_tile"),
                                      (6528, 80, "k_cg_tile"), (4097, 128, "k_cg_columns"),
                                      (6600, 80, "k_cg_columns"), (80000, 72, "k_cg_columns"),
                                      (80001, 72, "k_cg_solve (streaming)"),
                                      (130001, 80, "k_cg_solve (streaming)"),
                                      (400000, 100, "k_cg_columns")])
def test_choice(lib, m, N, want):
    assert lib.Plan(2 * m, m, N, 1, prec="fp64").solver_info()["solver"] == want


@pytest.mark.parametrize("m,N", [(1500, 70), (20000, 65), (80001, 66)])
def test_parity_cold_and_warm(lib, m, N):
    """Past the row-block solver's range and on either side of the streaming line."""
    import torch
    say(f"case: fp64 wide choice m={m} N={N}")
    p = W.random_problem(400, m, N, 1, seed=m, tol=1e-12)
    ref = O.enkf_reduced(p.Xf, p.idx, p.w, p.y, p.r, p.eps)["Xa"]   # the same analysis, N x N solve
    got = run(lib, p, "fp64", precond="diag_r", want_z=True, want_relres=True)
    assert got["status"] == 0 and rel(got["Xa"], ref) <= 1e-9 and got["relres"].max() <= 1e-10
    z0 = torch.as_tensor(got["Z"] * 1.001, device="cuda:0")
    warm = run(lib, p, "fp64", precond="diag_r", z0=z0)
    assert rel(warm["Xa"], ref) <= 1e-9


def test_captured_plan_sees_new_inputs(lib):
    """A captured call of the row-block solver, replayed on inputs changed in place."""
    import torch
    m, N = 2100, 90
    p, q = (W.random_problem(900, m, N, 2, seed=s, tol=1e-12) for s in (1, 2))
    plan = lib.Plan(900, m, N, 2, prec="fp64", tol=1e-12, maxit=2000)
    assert plan.solver_info()["solver"] == "k_cg_tile"
    d, dq = dev_problem(p, "fp64"), dev_problem(q, "fp64")
    out = torch.empty_like(d["Xf"])
    call = lambda: plan(d["Xf"], d["idx"], d["w"], d["y"], d["r"], d["eps"], out)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        call()
    for src in (d, dq, dev_problem(p, "fp64")):
        for key in d:
            d[key].copy_(src[key])
        g.replay()
        torch.cuda.synchronize()
        replayed = out.clone()
        out.zero_()
        call()
        torch.cuda.synchronize()
        assert torch.equal(out, replayed)
        ref = O.enkf_analysis(*(d[x].cpu().numpy() for x in ("Xf", "idx", "w", "y", "r", "eps")))
        assert rel(out.cpu().numpy(), ref["Xa"]) <= 1e-10
