"""Launches of more threads than HIP takes at once: the host's division of them (csrc/tc355_host.hpp, compiled by the system's C++
compiler) and one call that needs it."""
import ctypes
import os
import subprocess

import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def next_launch(tmp_path_factory):
    d = tmp_path_factory.mktemp("launch")
    (d / "launch.cpp").write_text('#include "tc355_host.hpp"\n'
                                  'extern "C" int64_t next_launch(int64_t left, int threads) { return tc355::next_launch(left, threads); }\n')
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_1802_04730_amd", "csrc"),
                    "-o", str(d / "launch.so"), str(d / "launch.cpp")], check=True)
    fn = ctypes.CDLL(str(d / "launch.so")).next_launch
    fn.restype = ctypes.c_int64
    return lambda left, threads: fn(ctypes.c_int64(left), ctypes.c_int(threads))


@pytest.mark.parametrize("threads", [256, 512, 1024])
@pytest.mark.parametrize("grid", [1, 8, (1 << 21) - 8, 1 << 21, (1 << 21) + 8, (1 << 23) + 1, 1 << 24, (1 << 24) + 8, 40265320, (1 << 31) - 1])
def test_every_workgroup_once_and_no_launch_too_large(next_launch, grid, threads):
    at = 0
    while at < grid:
        assert at % 8 == 0  # workgroups equal modulo 8 stay on one XCD
        n = next_launch(grid - at, threads)
        assert 0 < n and n * threads < 1 << 32
        at += n
    assert at == grid
    assert grid * threads > 1 << 31 or next_launch(grid, threads) == grid


@pytest.mark.gpu
def test_a_layer_of_2_24_tiles():
    """268435451 rows of 4 inputs, one output: 2^24 workgroups of 256 threads.  Small whole numbers: every value is exact."""
    from paper_1802_04730_amd import tc355 as tc
    batch = 268435451
    dims = (4, 1)
    I = torch.randint(-8, 9, (batch, 4), device="cuda", dtype=torch.int8).float()
    W = torch.tensor([[3.0, -2.0, 5.0, 1.0]], device="cuda")
    b = torch.tensor([7.0], device="cuda")
    O = torch.full((batch, 1), float("nan"), device="cuda")
    ws = torch.empty(max(256, tc.tc_mlp_fcrelu_workspace_bytes(batch, dims)), dtype=torch.uint8, device="cuda")
    tc.tc_mlp_fcrelu(I, [W], [b], [O], ws)
    torch.cuda.synchronize()
    assert tc.last_path() == "mlp:per_layer"
    for r in range(0, batch, 1 << 26):
        x = I[r:r + (1 << 26)]
        want = (x[:, 0] * 3 - x[:, 1] * 2 + x[:, 2] * 5 + x[:, 3] + 7).clamp_(min=0)
        assert torch.equal(O[r:r + (1 << 26), 0], want), r
