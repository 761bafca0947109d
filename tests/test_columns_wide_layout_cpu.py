"""Workspace of FP64 analyses with 64 < N <= 128: the column solver's buffers lie on
those of the other solvers, so that the size is that of the streaming solver's five m x N
arrays and its partial sums, for any m."""
import ctypes

import pytest

from paper_2606_19224_amd import binding


@pytest.mark.parametrize("N", [65, 72, 80, 96, 100, 127, 128])
def test_workspace_grows_by_five_arrays(N):
    size = lambda m: binding.workspace_bytes(m, m, N, 1, "fp64")
    for m in (200_000, 1_000_000, 2_000_000):   # the partial sums stop growing before
        assert abs(size(2 * m) - size(m) - 5 * 8 * N * m) <= 8 * 256


@pytest.mark.parametrize("N", [65, 72, 79, 80, 95, 96, 100, 128])
def test_layout_is_consistent(N):
    lib = binding.load()
    lib.cgd_layout_selfcheck.restype = ctypes.c_int
    for m in (1, 63, 64, 65, 1023, 1024, 1025, 1799, 1800, 4608, 79999, 80000, 80001, 130000,
              130001, 900_000, 4_194_304, 4_194_305):
        assert lib.cgd_layout_selfcheck(2 * m, m, N, 2, binding.PREC["fp64"]) == 0, m
