"""GPU parity of the batched matmul of small matrices at any alignment against the float64 oracle: one fp32 rounding of the
exact result (2.5e-7 on the metric, as for every fp64 kernel)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1802_04730_amd import inputs
from paper_1802_04730_amd.metric import parity_error

pytestmark = pytest.mark.gpu

TIGHT = 2.5e-7
GUARD = 64

# (B, N, M, K)
SHAPES = [
    (2, 1, 17, 2),           # X holds a single 16-byte piece
    (5, 1, 17, 1),
    (3, 17, 33, 7),          # the tensors end 1 and 1 elements into a piece
    (3, 15, 31, 9),          # 1 and 1 ... of another length
    (3, 13, 27, 5),          # 3 and 1
    (2, 17, 7, 15),          # 2 and 2
    (7, 17, 17, 31),
    (4000, 27, 61, 35),      # several jobs per wavefront; blocks of Z that share pieces
    (900, 9, 74, 12),        # five column tiles
    (300, 57, 19, 10),       # two tiles of rows per job
    (3000, 40, 40, 16),      # a reduction of one LDS bank's period
    (3000, 48, 48, 48),      # of three: rows of five column tiles would be mostly padding
    (1200, 58, 30, 12),      # results at any alignment as one stream
    (41, 60, 81, 32),        # long strips, few of them
    (300, 33, 65, 34),
    (200, 96, 96, 96),       # strips of columns: results row by row
    (60, 86, 92, 70),
    (40, 100, 100, 103),     # the longest reduction
    (40, 50, 99, 63),
    (40, 50, 17, 62),
    (64, 19, 83, 31),
]

# what stays on other kernels: (B, N, M, K), path
OTHERS = [
    ((5, 20, 30, 131), "tbmm:wave"),     # reductions too long for a strip in registers: loads of 1,
    ((3, 37, 33, 150), "tbmm:wave"),     # 2
    ((3, 17, 19, 300), "tbmm:wave"),     # and 4 elements
    ((3, 5, 200, 131), "tbmm:wave"),     # several strips of columns
    ((30, 9, 7, 5), "tbmm:wave"),        # nothing to stage
    ((300, 57, 16, 10), "tbmm:wave"),    # little to stage, one column tile
    ((40, 50, 99, 80), "tbmm:wave"),     # rows that share LDS banks: a wide result,
    ((40, 50, 16, 80), "tbmm:wave"),     # a narrow one
    ((60, 21, 101, 13), "tbmm:wave"),    # a wide result of a short odd reduction
    ((40, 120, 125, 68), "tbmm:tile"),   # 64 x 64 blocks: ragged ones, a reduction of two chunks and 4
    ((984, 53, 56, 88), "tbmm:tile"),    # three quarters full
    ((500, 26, 72, 26), "tbmm:lds"),
    ((130, 64, 64, 16), "tbmm:lds"),     # ... but short reductions stay with the strips
    ((700, 64, 60, 4), "tbmm:lds"),
    ((400, 48, 48, 48), "tbmm:lds"),     # enough long strips to hide their loads
    ((3000, 48, 56, 32), "tbmm:lds"),    # four of five column tiles
    ((5, 40, 40, 16), "tbmm:lds"),
    ((100, 8, 8, 128), "tbmm:lds"),      # reductions that are too long for the kernel of any alignment
    ((50, 4, 4, 256), "tbmm:lds"),
    ((1000, 17, 18, 112), "tbmm:lds"),
]


@pytest.mark.parametrize("shape,path", [(s, "tbmm:any") for s in SHAPES] + OTHERS)
def test_tbmm_any(shape, path, oracle_threads):
    from paper_1802_04730_amd import tc355 as tc
    B, N, M, K = shape
    X, Y = inputs.make_tbmm(B, N, M, K, seed=sum(shape))
    ref = oracle.tbmm(X, Y)
    buf = torch.full((ref.size + 2 * GUARD,), 777.0, device="cuda")
    Z = buf[GUARD:GUARD + ref.size].view(ref.shape)
    dev = lambda a: torch.from_numpy(a).cuda()
    tc.tc_tbmm(dev(X), dev(Y), Z)
    torch.cuda.synchronize()
    assert tc.last_path() == path
    err = parity_error(Z.cpu().numpy().astype(np.float64), ref)
    print("tbmm %s: parity error %.3e" % (shape, err), flush=True)
    assert err <= TIGHT
    assert bool((buf[:GUARD] == 777.0).all()) and bool((buf[GUARD + ref.size:] == 777.0).all())


@pytest.mark.parametrize("shape", [(3, 17, 33, 7), (3, 17, 33, 11), (5, 40, 40, 16), (41, 60, 81, 32), (4, 96, 90, 50)])
def test_tbmm_keeps_infinities_in_their_rows(shape, oracle_threads):
    """Slots past K of a last step hold the next row's data: an Inf there reaches nothing."""
    from paper_1802_04730_amd import tc355 as tc
    B, N, M, K = shape
    X, Y = (np.abs(a) + np.float32(0.1) for a in inputs.make_tbmm(B, N, M, K, seed=4))
    X[1, N - 2, 0] = np.inf
    Y[B - 1, M - 1, K - 1] = np.inf
    ref = oracle.tbmm(X, Y)
    Z = torch.empty(ref.shape, device="cuda")
    tc.tc_tbmm(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(), Z)
    got = Z.cpu().numpy()
    assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and np.isposinf(ref).any() and not np.isnan(got).any()
