"""GPU parity of the Kronecker layer of any extents (operands staged in LDS) against the float64 oracle: one fp32 rounding
of the exact result (2.5e-7 on the metric, as for every fp64 kernel)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1802_04730_amd import inputs
from paper_1802_04730_amd.metric import parity_error

pytestmark = pytest.mark.gpu

TIGHT = 2.5e-7
GUARD = 64

# (B, I, K, J, L)
SHAPES = [
    (1, 2, 2, 2, 2),           # the smallest that are staged: a partial group and a partial tile only
    (3, 1, 5, 1, 3),
    (2, 16, 16, 16, 16),       # whole tiles and groups, nothing partial
    (5, 17, 17, 17, 17),       # one more of each
    (7, 15, 31, 33, 31),
    (40, 79, 89, 29, 74),      # fewer batch elements than compute units: the l tiles of a row block are split
    (3, 9, 84, 55, 55),        # one row block, its four l tiles on four wavefronts
    (2, 20, 7, 30, 130),       # nine l tiles on four wavefronts
    (300, 48, 50, 75, 36),     # one batch element per stage, more stages than workgroups are resident
    (2100, 18, 21, 40, 23),    # four batch elements per stage, the last stage with fewer
    (3000, 9, 10, 11, 13),     # eight per stage; rows of zeros between them
    (4, 100, 100, 100, 100),   # fp32 in LDS
    (2, 64, 32, 128, 48),      # eight column tiles
    (2, 33, 10, 140, 20),      # two blocks of columns
    (2, 150, 12, 20, 18),      # two blocks of rows
    (1, 40, 300, 24, 40),      # a long first reduction
    (4, 128, 128, 128, 128),   # one block of rows does not fit LDS
    (515, 40, 700, 9, 20),     # ... with more batch elements than two workgroups per compute unit
]


def run(tc, W1, W2, X, path="kron:tile"):
    shape = (X.shape[0], W1.shape[0], W2.shape[0])
    size = int(np.prod(shape))
    buf = torch.full((size + 2 * GUARD,), 777.0, device="cuda")
    Y = buf[GUARD:GUARD + size].view(shape)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    tc.tc_kron(dev(W1), dev(W2), dev(X), Y)
    torch.cuda.synchronize()
    assert tc.last_path() == path
    assert bool((buf[:GUARD] == 777.0).all()) and bool((buf[GUARD + size:] == 777.0).all())
    return Y.cpu().numpy()


@pytest.mark.parametrize("shape", SHAPES)
def test_kron_any(shape, oracle_threads):
    from paper_1802_04730_amd import tc355 as tc
    W1, W2, X = inputs.make_kron(*shape, seed=sum(shape))
    err = parity_error(run(tc, W1, W2, X).astype(np.float64), oracle.kron(W1, W2, X))
    print("kron %s: parity error %.3e" % (shape, err), flush=True)
    assert err <= TIGHT


@pytest.mark.parametrize("shape", [
    (3, 20, 1, 30, 17),        # nothing to contract first ...
    (3, 17, 20, 70, 1),        # ... or second
    (2, 37, 200, 41, 203),     # one batch element of X is larger than LDS
    (5, 33, 18, 70, 1200),     # 16 columns of W2 and X are
])
def test_kron_beyond_lds(shape, oracle_threads):
    from paper_1802_04730_amd import tc355 as tc
    W1, W2, X = inputs.make_kron(*shape, seed=sum(shape))
    assert parity_error(run(tc, W1, W2, X, "kron:wave").astype(np.float64), oracle.kron(W1, W2, X)) <= TIGHT


@pytest.mark.parametrize("shape", [(3, 18, 21, 19, 23), (40, 18, 21, 19, 55)])
def test_kron_keeps_infinities_out_of_the_padding(shape, oracle_threads):
    """The zeros of partial steps multiply nothing but zeros: an Inf in any operand reaches the outputs that read it only."""
    from paper_1802_04730_amd import tc355 as tc
    for where in range(3):
        ops = [np.abs(a) + 0.01 for a in inputs.make_kron(*shape, seed=3)]
        ops[where][tuple(n - 1 for n in ops[where].shape)] = np.inf
        W1, W2, X = (a.astype(np.float32) for a in ops)
        ref = oracle.kron(W1, W2, X)
        got = run(tc, W1, W2, X)
        assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and 0 < np.isposinf(ref).sum() < ref.size
        assert not np.isnan(got).any()
