"""Which variant of a kernel the shapes of the GPU tests take: the library's own choice (csrc/kron_tile_plan.hpp,
csrc/gemm_direct_plan.hpp, compiled by the system's C++ compiler) for 256 compute units.  All variants report one path, so a line
that moves would take the coverage with it unseen."""
import ctypes
import os
import subprocess

import pytest

import test_gpu_gemm_direct
import test_gpu_kron_order

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CUS = 256


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("plans") / "plans.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_1802_04730_amd", "csrc"),
                    "-o", lib, os.path.join(ROOT, "tests", "plans_host.cpp")], check=True)
    return ctypes.CDLL(lib)


def kron(plans, shape):
    out = (ctypes.c_int64 * 9)()
    assert plans.kron(*[ctypes.c_int64(x) for x in shape], ctypes.c_int(CUS), out), shape
    return dict(zip(("second", "wide", "nb", "lsp", "i_blocks", "j_blocks", "tj", "stages", "workgroups"), out))


def test_kron_orders(plans):
    for shape in test_gpu_kron_order.SECOND + test_gpu_kron_order.POISONED:
        assert kron(plans, shape)["second"], shape
    for shape in test_gpu_kron_order.FIRST:
        assert not kron(plans, shape)["second"], shape


# What each shape of SECOND is there for, as far as the plan says it
SAID = {
    (300, 64, 17, 16, 96): dict(lsp=2, wide=1),
    (300, 65, 31, 17, 95): dict(lsp=1, tj=5),
    (2100, 40, 9, 10, 97): dict(nb=5, stages=420),
    (2, 120, 10, 40, 1000): dict(wide=0, tj=8),
    (1, 29, 4, 61, 85): dict(lsp=1, j_blocks=4),
    (1, 42, 3, 73, 56): dict(lsp=1, tj=3),
    (300, 41, 40, 25, 23): dict(lsp=1),
    (1, 30, 35, 45, 38): dict(lsp=2),
    (1, 24, 31, 21, 43): dict(lsp=2),
    (1, 150, 9, 69, 22): dict(i_blocks=2, j_blocks=5),
    (253, 153, 19, 28, 22): dict(i_blocks=2, nb=2),
    (523, 22, 65, 15, 226): dict(wide=0, lsp=2, nb=2, stages=262, workgroups=256),
    (1181, 24, 90, 5, 83): dict(wide=1, lsp=2, nb=2, stages=591, workgroups=256),
    (258, 19, 110, 47, 282): dict(wide=0, lsp=4, j_blocks=3, stages=258, workgroups=85),
}


def test_kron_variants(plans):
    assert set(SAID) == set(test_gpu_kron_order.SECOND)
    for shape, said in SAID.items():
        plan = kron(plans, shape)
        assert {k: plan[k] for k in said} == said, (shape, plan)


# Tiles of 16 x 16 per workgroup and wavefronts
DIRECT = {
    (17, 33, 4): (1, 1, 4), (17, 33, 5): (1, 1, 4), (17, 33, 6): (1, 1, 4), (17, 33, 19): (1, 1, 4), (1, 16, 161): (1, 1, 4), (130, 1031, 261): (1, 1, 4),
    (40, 300, 259): (1, 1, 8), (128, 1030, 515): (1, 1, 8), (5, 7, 1021): (1, 1, 16), (20, 100, 1003): (1, 1, 16),
    (300, 257, 160): (1, 2, 8), (300, 257, 163): (1, 2, 8), (700, 999, 160): (2, 2, 4), (700, 999, 161): (2, 2, 4),
}


@pytest.mark.parametrize("size", [4, 8])
def test_split_reduction_variants(plans, size):
    assert set(DIRECT) == set(test_gpu_gemm_direct.SHAPES)
    out = (ctypes.c_int * 3)()
    for (N, M, K), variant in DIRECT.items():
        plans.direct(ctypes.c_int64(N), ctypes.c_int64(M), ctypes.c_int64(K), ctypes.c_int(size), ctypes.c_int(CUS), out)
        assert tuple(out) == variant, (N, M, K)
