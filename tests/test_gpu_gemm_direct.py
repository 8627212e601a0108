"""GPU parity of the split-reduction kernel (operands loaded straight to LDS): each of its tile and wavefront counts on fp32 rows
(tc_tbmm with B = 1) and on fp64 activations (the second layer of a chain), at ragged extents and reductions that end inside a
step, against the float64 oracle: one fp32 rounding of the exact result (2.5e-7 on the metric, as for every fp64 kernel)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1802_04730_amd import inputs
from paper_1802_04730_amd.metric import parity_error

pytestmark = pytest.mark.gpu

TIGHT = 2.5e-7
GUARD = 64

# (N, M, K)
SHAPES = [
    (17, 33, 4), (17, 33, 5), (17, 33, 6), (17, 33, 19),  # less than a step, a step and a part: four wavefronts, some without work
    (1, 16, 161), (130, 1031, 261),                       # four wavefronts
    (40, 300, 259), (128, 1030, 515),                     # eight
    (5, 7, 1021), (20, 100, 1003),                        # sixteen
    (300, 257, 160), (300, 257, 163),                     # 1 x 2 tiles, whole steps and a part of one
    (700, 999, 160), (700, 999, 161),                     # 2 x 2 tiles
]


def guarded(*shape):
    size = int(np.prod(shape))
    buf = torch.full((size + 2 * GUARD,), 777.0, device="cuda")
    return buf, buf[GUARD:GUARD + size].view(shape)


def clean(buf):
    return bool((buf[:GUARD] == 777.0).all()) and bool((buf[-GUARD:] == 777.0).all())


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


@pytest.mark.parametrize("shape", SHAPES[1:])  # (a plain product of 4 takes the strips in registers)
def test_fp32_rows(shape, oracle_threads):
    from paper_1802_04730_amd import tc355 as tc
    N, M, K = shape
    X, Y = inputs.make_tbmm(1, N, M, K, seed=N + M + K)
    buf, Z = guarded(1, N, M)
    tc.tc_tbmm(dev(X), dev(Y), Z)
    torch.cuda.synchronize()
    assert tc.last_path() == "tbmm:splitk"
    err = parity_error(Z.cpu().numpy().astype(np.float64), oracle.tbmm(X, Y))
    print("product %s: parity error %.3e" % (shape, err), flush=True)
    assert err <= TIGHT and clean(buf)


@pytest.mark.parametrize("shape", SHAPES)
def test_fp64_activations(shape, oracle_threads):
    from paper_1802_04730_amd import tc355 as tc
    batch, M, K = shape
    dims = (9, K, M)
    I, Ws, bs = inputs.make_mlp(batch, dims, seed=batch + K, w_std=0.1)
    ref = oracle.mlp_fcrelu(I, Ws, bs)
    outs = [guarded(batch, d) for d in dims[1:]]
    ws = torch.full((tc.tc_mlp_fcrelu_workspace_bytes(batch, dims),), 0xCD, dtype=torch.uint8, device="cuda")
    tc.tc_mlp_fcrelu(dev(I), [dev(w) for w in Ws], [dev(b) for b in bs], [o for _, o in outs], ws)
    torch.cuda.synchronize()
    assert tc.last_path() == "mlp:per_layer"
    for (buf, o), r in zip(outs, ref):
        err = parity_error(o.cpu().numpy().astype(np.float64), r)
        print("chain %s: parity error %.3e" % (shape, err), flush=True)
        assert err <= TIGHT and clean(buf)


@pytest.mark.parametrize("shape", [(17, 33, 7), (40, 300, 259), (300, 257, 163), (700, 999, 161)])
def test_infinities_stay_where_they_are(shape, oracle_threads):
    """What a group of 4 that is moved back shares with the one before counts once, and as zero in both operands elsewhere."""
    from paper_1802_04730_amd import tc355 as tc
    N, M, K = shape
    X, Y = (np.abs(a) + 0.1 for a in inputs.make_tbmm(1, N, M, K, seed=9))
    for k in (0, K // 2, K - 4, K - 1):
        X[0, k % N, k] = np.inf
        Y[0, (k + 1) % M, k] = np.inf
    X, Y = X.astype(np.float32), Y.astype(np.float32)
    ref = oracle.tbmm(X, Y)
    buf, Z = guarded(1, N, M)
    tc.tc_tbmm(dev(X), dev(Y), Z)
    got = Z.cpu().numpy()
    assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and not np.isnan(got).any() and clean(buf)
