"""FP32 batches take any number of rows, as FP64 ones do (the group solver's index
arithmetic ends at 2^22 rows; the per-member solver takes over there)."""
import ctypes

import pytest

from paper_2606_19224_amd import binding


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("m", [1 << 22, (1 << 22) + 1, 6_000_000])
def test_many_rows_are_accepted(prec, m):
    lib = binding.load()
    arr = (binding.CProblem * 1)(binding.CProblem(m, m, 8, 1, *([None] * 8), 0, 0))
    f = lib.cgd_enkf_batched_workspace_bytes
    f.argtypes = [ctypes.c_int, ctypes.POINTER(binding.CProblem), ctypes.c_int]
    f.restype = ctypes.c_size_t
    assert f(1, arr, binding.PREC[prec]) > m * 8 * 4
