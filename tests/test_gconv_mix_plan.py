"""Staging of the shape-generic grouped convolution, walked on the host with the kernel's own plan and index arithmetic
(csrc/gconv_mix_plan.hpp, compiled by the system's C++ compiler): every element that a stage contracts is staged, from the
right place, and nothing outside the input is read."""
import ctypes
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("walk") / "walk.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_1802_04730_amd", "csrc"),
                    "-o", lib, os.path.join(ROOT, "tests", "gconv_mix_walk.cpp")], check=True)
    fn = ctypes.CDLL(lib).walk
    fn.restype = ctypes.c_int64
    plan = (ctypes.c_int * 6)()

    def call(shape, cus=256):
        faults = fn(*[ctypes.c_int(x) for x in shape], ctypes.c_int(cus), plan)
        return faults, dict(zip(("imgs", "chunks", "jobs", "grid", "pblocks", "alike"), plan))
    return call


# Several images per job and several chunks of channels: the last chunk of a full block of images and the first chunk of
# the last block are as many units, laid out differently.  (N, G, C, F, H, W, KH, KW)
ALIKE = [(33, 63, 42, 2, 9, 17, 3, 3), (39, 62, 40, 3, 11, 11, 3, 3), (62, 54, 30, 3, 18, 6, 3, 3)]


@pytest.mark.parametrize("shape", ALIKE)
def test_stages_of_as_many_units_in_another_layout(walk, shape):
    faults, plan = walk(shape)
    assert plan["imgs"] > 1 and plan["chunks"] > 1 and plan["jobs"] > plan["grid"] and plan["alike"] > 0, plan
    assert faults == 0, plan


def test_random_plans(walk):
    """Few compute units, so that workgroups walk long runs of jobs."""
    rng = random.Random(7)
    seen = dict(alike=0, several=0, chunks=0, blocks=0)
    for _ in range(400):
        k = rng.choice([1, 2, 3, 3, 5])
        h, w = (rng.randint(k, 12), rng.randint(k, 12)) if rng.random() < 0.6 else (rng.randint(k, 40), rng.randint(k, 40))
        shape = (rng.randint(1, 9), rng.randint(1, 3), rng.randint(1, 100), rng.randint(1, 70), h, w, k, k)
        faults, plan = walk(shape, cus=rng.randint(1, 4))
        assert faults <= 0, (shape, plan)
        if faults == 0:
            seen["alike"] += plan["alike"]
            seen["several"] += plan["imgs"] > 1
            seen["chunks"] += plan["chunks"] > 1
            seen["blocks"] += plan["pblocks"] > 1
    assert min(seen.values()) > 0, seen
