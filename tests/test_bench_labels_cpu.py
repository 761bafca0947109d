"""What bench.py says about a solver: the kernel, its peak's unit and its bytes, for the
FP64 forms past N = 64 and for batches.  No GPU needed."""
from types import SimpleNamespace

import numpy as np
import pytest

import bench


def _label(solver, prec, m, N, n=8000, rows=128, wgs=8, it=10):
    return bench.solver_roofline({"solver": solver, "rows_per_block": rows, "workgroups": wgs},
                                 SimpleNamespace(prec=prec), m, N, 1, n, np.array([it]))


def test_fp64_row_block_solver_is_named_for_what_it_is():
    by, fl, kernel, limiter, mfma = _label("k_cg_tile", "fp64", 2000, 100)
    assert kernel.startswith("k_cg_tile64 ") and "FP64 MFMA" in kernel and "16 members" in kernel
    assert mfma and "FP32" not in kernel + limiter
    assert _label("k_cg_tile", "fp32", 2000, 100)[2].startswith("k_cg_tile<float>")


@pytest.mark.parametrize("solver", ["k_cg_columns", "k_cg_tile"])
def test_fp64_solvers_past_64_members_do_not_update(solver):
    # the update is a launch of its own: the timed bytes do not depend on n
    a, b = (_label(solver, "fp64", 1000, 100, n=n)[0][0] for n in (2000, 200000))
    assert a == b
    small = [_label("k_cg_columns", "fp64", 1000, 64, n=n)[0][0] for n in (2000, 200000)]
    assert small[1] - small[0] == 2.0 * 198000 * 64 * 8


def test_few_rows_are_named_for_the_one_wave_solver():
    name = lambda *a: _label("k_cg_columns", *a)[2].split("<")[0]
    assert name("fp64", 20, 20) == name("fp32", 128, 64) == name("fp64", 64, 64) == "k_cg_columns_small"
    assert name("fp64", 65, 64) == name("fp32", 129, 20) == name("mixed", 20, 20) == "k_cg_columns"


def test_batched_bytes_count_s_once_per_group():
    p = SimpleNamespace(m=1000, N=64)
    one, four = (bench.batched_solve_bytes(p, 10, g) for g in (1, 4))
    # S and diag(R) per pass and member or group, r and p of every member
    assert one == 4.0 * 64 * 1000 * (11 * 65 + 41)
    assert four == 4.0 * 16 * 1000 * (11 * 65 + 4 * 41)
    assert bench.batched_solve_flops(p, 0) == 2.0 * 1000 * 64 * 64
