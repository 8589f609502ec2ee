"""The ILU kernel the benchmark reports is the one a handle of that size runs."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


@pytest.mark.parametrize("args,name", [
    ((False, 0, "fp64", 0, 5632), "k_ilu_jacobi"),
    ((False, 0, "fp64", 0, 5633), "k_ilu_jacobi_blocks"),
    ((False, 0, "fp64", 1, 4097), "k_ilu_jacobi_blocks"),
    ((False, 0, "fp16", 1, 8192), "k_ilu_jacobi"),
    ((False, 0, "fp16", 1, 8193), "k_ilu_jacobi_blocks"),
    ((False, 1, "fp32", 0, 5632), "k_ilu_jacobi_phased"),
    ((False, 1, "fp32", 0, 9200), "k_ilu_jacobi_blocks"),
    ((False, 2, "fp64", 0, 100), "k_ilu_jacobi_blocks"),
    ((False, 4, "fp64", 0, 100), "k_ilu_jacobi_hold"),
    ((True, 0, "fp32", 1, 100), "k_ilu_jacobi_hold"),
    ((False, 0, "fp64", 2, 100), "k_ilu_jacobi_generic"),
])
def test_ilu_kernel_names(args, name):
    assert bench.ilu_kernel_name(*args) == name
