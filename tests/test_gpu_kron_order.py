"""GPU parity of the Kronecker layer where the second factor is applied first (fewer multiply-adds that way), at the edges of
its tiles: one fp32 rounding of the exact result (2.5e-7 on the metric, as for every fp64 kernel)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1802_04730_amd import inputs
from paper_1802_04730_amd.metric import parity_error

pytestmark = pytest.mark.gpu

TIGHT = 2.5e-7
GUARD = 64

# (B, I, K, J, L): I and L large against K and J.  tests/test_variant_plans.py holds them to what is said here.
SECOND = [
    (300, 64, 17, 16, 96),    # one row of k in the second tile; whole groups of l; two wavefronts per tile
    (300, 65, 31, 17, 95),    # partial everything; one column of the second tile of j
    (2100, 40, 9, 10, 97),    # several batch elements per stage, the last stage with fewer
    (2, 120, 10, 40, 1000),   # fp32 in LDS, eight accumulators
    (1, 29, 4, 61, 85),       # one batch element; a tile of 4 k; l in 5 groups and a partial one of 5; blocks of rows
    (1, 42, 3, 73, 56),       # a tile of 3 k
    (300, 41, 40, 25, 23),    # three tiles of k: a pair and one
    (1, 30, 35, 45, 38),      # three tiles of k split over two wavefronts
    (1, 24, 31, 21, 43),      # two tiles of k split over two wavefronts, the second one partial
    (1, 150, 9, 69, 22),      # two blocks of columns of the result, five of its rows
    (253, 153, 19, 28, 22),   # two blocks of columns, two batch elements per stage, the last stage with one
    (523, 22, 65, 15, 226),   # partial sums where X lay, and then X again: six workgroups take two stages; fp32
    (1181, 24, 90, 5, 83),    # the same in fp64, two and three stages
    (258, 19, 110, 47, 282),  # the same with four wavefronts per tile, blocks of rows, fp32
]
# ... and where the first one goes first all the same
FIRST = [
    (40, 100, 16, 8, 100),
    (7, 33, 5, 3, 131),
    (3, 128, 33, 9, 66),
    (2, 140, 20, 33, 90),
    (1, 96, 64, 16, 200),
]
POISONED = [(300, 65, 31, 17, 95), (700, 18, 37, 12, 61), (300, 151, 17, 4, 18)]  # (partial tiles of k, second factor first)


def both(shape, poison=False):
    from paper_1802_04730_amd import tc355 as tc
    W1, W2, X = inputs.make_kron(*shape, seed=sum(shape))
    if poison:  # an infinity in the last row of each operand: only what reads it may see it
        W1, W2, X = (np.abs(a) + 0.01 for a in (W1, W2, X))
        W1[-1, -1] = np.inf
        X[-1, -1, -1] = np.inf
    W1, W2, X = (np.ascontiguousarray(a, dtype=np.float32) for a in (W1, W2, X))
    B, I, K, J, L = shape
    buf = torch.full((B * I * J + 2 * GUARD,), 777.0, device="cuda")
    Y = buf[GUARD:GUARD + B * I * J].view(B, I, J)
    dev = lambda a: torch.from_numpy(a).cuda()
    tc.tc_kron(dev(W1), dev(W2), dev(X), Y)
    torch.cuda.synchronize()
    assert tc.last_path() == "kron:tile"
    assert bool((buf[:GUARD] == 777.0).all()) and bool((buf[GUARD + B * I * J:] == 777.0).all())
    return Y.cpu().numpy(), oracle.kron(W1, W2, X)


@pytest.mark.parametrize("shape", SECOND + FIRST)
def test_kron_second_factor_first(shape, oracle_threads):
    got, ref = both(shape)
    err = parity_error(got.astype(np.float64), ref)
    print("kron %s: parity error %.3e" % (shape, err), flush=True)
    assert err <= TIGHT


@pytest.mark.parametrize("shape", POISONED)
def test_kron_second_factor_first_keeps_infinities_apart(shape, oracle_threads):
    got, ref = both(shape, poison=True)
    finite = np.isfinite(ref)
    assert np.array_equal(np.isfinite(got), finite)
    assert parity_error(got[finite].astype(np.float64), ref[finite]) <= TIGHT


@pytest.mark.parametrize("shape", [SECOND[1], FIRST[0]])
@pytest.mark.parametrize("factor", [1, 2])
def test_infinity_in_a_factor(shape, factor):
    """The factor that goes first meets the elements of X one by one (Inf times a zero is NaN), the other one their sums."""
    from paper_1802_04730_amd import tc355 as tc
    B, I, K, J, L = shape
    W = [np.abs(a) + 0.01 for a in inputs.make_kron(*shape, seed=5)]
    W[factor - 1][0, 0] = np.inf
    W[2][0, 0, 0] = 0.0
    W1, W2, X = (torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda() for a in W)
    Y = torch.empty((B, I, J), device="cuda")
    tc.tc_kron(W1, W2, X, Y)
    assert tc.last_path() == "kron:tile"
    first = 2 if shape in SECOND else 1  # the factor that goes first
    hit = Y[:, 0, :] if factor == 1 else Y[:, :, 0]  # what reads the infinity
    assert bool(hit[1:].isposinf().all())
    assert bool((hit[0].isnan() if factor == first else hit[0].isposinf()).all())
    rest = Y[:, 1:, :] if factor == 1 else Y[:, :, 1:]
    assert bool(rest.isfinite().all())
