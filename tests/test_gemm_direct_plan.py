"""The loads of the split-reduction kernel, walked on the host with the kernel's own index arithmetic (csrc/gemm_direct_plan.hpp,
compiled by the system's C++ compiler)."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("walk") / "walk.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_1802_04730_amd", "csrc"),
                    "-o", lib, os.path.join(ROOT, "tests", "gemm_direct_walk.cpp")], check=True)
    return ctypes.CDLL(lib)


@pytest.mark.parametrize("size", [4, 8])
@pytest.mark.parametrize("K", list(range(4, 36)) + [100, 1000, 1021, 65537])
def test_loads_stay_inside_the_operand(walk, K, size):
    """At every reduction that ends inside a step, up to the most rows that the kernel is given."""
    loads, reaches = walk.walk_loads, walk.reaches
    loads.restype = ctypes.c_int64
    most = ((1 << 32) - 1) // (K * size)
    while not reaches(ctypes.c_int64(most), K, size):
        most -= 1
    assert (most + 1) * K * size >= (1 << 32) - 256  # (all but the last few hundred bytes of 4 GiB)
    for rows in (1, 2, 17, most // 2, most - 1, most):
        assert loads(ctypes.c_int64(rows), K, size) == 0, rows


@pytest.mark.parametrize("rows,K", [(268435455, 4), (214748364, 5), (178956970, 6), (153391689, 7), (119304647, 9), (97612893, 11)])
def test_rows_that_would_be_read_in_front_of_the_operand_are_refused(walk, rows, K):
    walk.walk_loads.restype = ctypes.c_int64
    assert rows * K * 4 < 1 << 32 and walk.walk_loads(ctypes.c_int64(rows), K, 4) > 0
    assert not walk.reaches(ctypes.c_int64(rows), K, 4)
