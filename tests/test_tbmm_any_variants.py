"""Every tile and way out of the batched matmul at any alignment, with one to four batch elements per workgroup: which one a shape takes
(the library's own choice in csrc/tbmm_any_plan.hpp, compiled by the system's C++ compiler, for 256 compute units) and, on the GPU, its
parity with the float64 oracle: one fp32 rounding of the exact result (2.5e-7 on the metric, as for every fp64 kernel)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest
import torch

import oracle
from paper_1802_04730_amd import inputs
from paper_1802_04730_amd.metric import parity_error

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TIGHT = 2.5e-7
GUARD = 64

# (B, N, M, K): tiles per wavefront, wavefronts of rows and columns, batch elements per workgroup, results from the registers, strips
VARIANTS = {
    (2, 1, 3, 10): ((1, 1), (1, 1), 1, 1, (1, 1)),  # a workgroup of one wavefront
    (3, 3, 73, 2): ((1, 1), (1, 3), 1, 1, (1, 2)),
    (276, 1, 1, 38): ((1, 1), (1, 1), 2, 1, (1, 1)),  # two batch elements per workgroup
    (1564, 16, 60, 44): ((1, 1), (1, 4), 1, 0, (1, 1)),
    (2, 32, 36, 28): ((1, 1), (2, 2), 1, 1, (1, 2)),  # K a multiple of 4: permuted pieces; the second strip of columns is 4 rows
    (181, 101, 97, 2): ((1, 2), (1, 4), 1, 0, (7, 1)),  # strips of rows, the last one of 5, that stay one block of Z
    (291, 56, 93, 15): ((1, 2), (4, 1), 1, 0, (1, 3)),  # strips of columns: results row by row through LDS
    (338, 47, 97, 4): ((1, 2), (1, 4), 1, 0, (3, 1)),
    (112, 51, 99, 76): ((1, 2), (4, 2), 1, 1, (1, 2)),
    (364, 107, 39, 1): ((1, 3), (4, 1), 1, 0, (2, 1)),
    (343, 48, 93, 8): ((1, 3), (3, 1), 1, 0, (1, 2)),
    (1590, 11, 87, 2): ((1, 3), (1, 2), 2, 0, (1, 1)),
    (284, 33, 69, 3): ((1, 5), (3, 1), 1, 1, (1, 1)),
    (1125, 20, 71, 4): ((1, 5), (2, 1), 2, 0, (1, 1)),
    (194, 21, 66, 1): ((2, 1), (1, 5), 1, 1, (1, 1)),
    (145, 100, 107, 10): ((2, 1), (4, 1), 1, 0, (1, 7)),  # strips of 16 columns
    (44, 98, 99, 84): ((2, 1), (4, 2), 1, 1, (1, 4)),  # 8 wavefronts
    (1478, 52, 4, 8): ((2, 1), (2, 1), 2, 1, (1, 1)),
    (119, 97, 104, 2): ((2, 2), (4, 2), 1, 1, (1, 2)),
    (1059, 31, 50, 4): ((2, 2), (1, 2), 2, 0, (1, 1)),
    (403, 99, 39, 2): ((2, 3), (4, 1), 1, 0, (1, 1)),
    (345, 80, 88, 76): ((2, 3), (3, 1), 1, 1, (1, 2)),
    (117, 66, 68, 5): ((3, 1), (2, 3), 1, 1, (1, 2)),
    (328, 65, 71, 4): ((3, 1), (2, 2), 1, 0, (1, 3)),
    (807, 33, 60, 1): ((3, 2), (1, 2), 2, 0, (1, 1)),
    (341, 67, 102, 64): ((3, 2), (2, 2), 1, 1, (1, 2)),
    (270, 33, 70, 2): ((3, 3), (1, 2), 2, 1, (1, 1)),
    (305, 70, 69, 4): ((3, 3), (2, 2), 1, 1, (1, 1)),
    (387, 95, 41, 4): ((3, 3), (2, 1), 2, 0, (1, 1)),
    # three and four batch elements per workgroup, the last one short of some
    (2275, 8, 38, 13): ((1, 3), (1, 1), 3, 1, (1, 1)),
    (2276, 8, 38, 13): ((1, 3), (1, 1), 3, 1, (1, 1)),
    (11861, 3, 33, 35): ((1, 3), (1, 1), 4, 1, (1, 1)),
    (3001, 7, 45, 60): ((1, 3), (1, 1), 4, 1, (1, 1)),
    (4002, 9, 45, 60): ((1, 3), (1, 1), 4, 0, (1, 1)),
    (3001, 20, 30, 33): ((2, 2), (1, 1), 4, 0, (1, 1)),
    (3251, 41, 40, 51): ((3, 3), (1, 1), 4, 0, (1, 1)),
}


def test_variant_of_each_shape(tmp_path):
    src, lib = tmp_path / "plan.cpp", str(tmp_path / "plan.so")
    src.write_text('#include "tbmm_any_plan.hpp"\n'
                   'extern "C" int plan(int64_t B, int64_t N, int64_t M, int64_t K, int64_t* o) {\n'
                   '  tc355::TbmmAnyPlan p{};\n'
                   '  if (!tc355::choose_tbmm_any(B, N, M, K, 256, &p)) return 0;\n'
                   '  const int64_t v[10] = {p.tn, p.tm, p.gn, p.gm, p.nb, p.direct, p.strips_n, p.strips_m, p.groups, p.lds};\n'
                   '  for (int i = 0; i < 10; i++) o[i] = v[i];\n'
                   '  return 1;\n}\n')
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_1802_04730_amd", "csrc"),
                    "-o", lib, str(src)], check=True)
    plan = ctypes.CDLL(lib).plan
    o = (ctypes.c_int64 * 10)()
    for shape, said in VARIANTS.items():
        assert plan(*[ctypes.c_int64(x) for x in shape], o)
        assert ((o[0], o[1]), (o[2], o[3]), o[4], o[5], (o[6], o[7])) == said, shape
    rng = np.random.default_rng(5)
    for _ in range(3000):  # what the kernel takes for granted of any plan
        B, N, M, K = (int(x) for x in (rng.integers(1, 1 << rng.integers(1, 20)), rng.integers(1, 400), rng.integers(1, 400), rng.integers(1, 104)))
        if not plan(*[ctypes.c_int64(x) for x in (B, N, M, K)], o):
            continue
        tn, tm, gn, gm, nb, direct, sn, sm, groups, lds = o
        assert 1 <= gn * gm * nb <= 8 and (nb == 1 or sn * sm == 1)
        assert sn * 16 * tn * gn >= N > (sn - 1) * 16 * tn * gn and sm * 16 * tm * gm >= M > (sm - 1) * 16 * tm * gm
        assert groups == (-(-B // nb) if sn * sm == 1 else B * sn * sm) < 1 << 31
        rows, cols, unit = min(16 * tn * gn, N), min(16 * tm * gm, M), 64 if K % 4 == 0 else 4
        need = (-(-nb * rows * K // unit) + -(-nb * cols * K // unit)) * 4 * unit  # both strips, in whole (groups of 16) pieces
        assert max(need, 0 if direct else 4 * (nb * rows * cols + 3)) <= lds <= 160 * 1024


@pytest.mark.gpu
@pytest.mark.parametrize("shape", list(VARIANTS))
def test_variants(shape, oracle_threads):
    from paper_1802_04730_amd import tc355 as tc
    B, N, M, K = shape
    X, Y = inputs.make_tbmm(B, N, M, K, seed=sum(shape))
    ref = oracle.tbmm(X, Y)
    buf = torch.full((ref.size + 2 * GUARD,), 777.0, device="cuda")
    Z = buf[GUARD:GUARD + ref.size].view(ref.shape)
    tc.tc_tbmm(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(), Z)
    torch.cuda.synchronize()
    assert tc.last_path() == "tbmm:any"
    err = parity_error(Z.cpu().numpy().astype(np.float64), ref)
    print("tbmm %s: parity error %.3e" % (shape, err), flush=True)
    assert err <= TIGHT
    assert bool((buf[:GUARD] == 777.0).all()) and bool((buf[GUARD + ref.size:] == 777.0).all())
