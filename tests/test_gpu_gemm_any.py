"""GPU parity of single products and fully connected layers of any width (rows at any 4-byte alignment, reductions that are
no multiple of a load or a chunk) against the float64 oracle: one fp32 rounding of the exact result (2.5e-7 on the metric,
as for every fp64 kernel)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1802_04730_amd import inputs
from paper_1802_04730_amd.metric import parity_error

pytestmark = pytest.mark.gpu

TIGHT = 2.5e-7
GUARD = 64


def guarded(shape):
    size = int(np.prod(shape))
    buf = torch.full((size + 2 * GUARD,), 777.0, device="cuda")
    return buf, buf[GUARD:GUARD + size].view(shape)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def clean(buf):
    return bool((buf[:GUARD] == 777.0).all()) and bool((buf[-GUARD:] == 777.0).all())


# (N, M, K), kernel
PRODUCTS = [
    ((3, 5, 3), "tbmm:wave"),           # too short for a 16-byte piece
    ((13, 11, 13), "tbmm:wave"),
    ((17, 33, 4), "tbmm:lds"),
    ((17, 33, 5), "tbmm:splitk"),       # the last piece moved back over the one before
    ((17, 33, 7), "tbmm:splitk"),
    ((33, 17, 127), "tbmm:splitk"),     # one short chunk
    ((33, 17, 128), "tbmm:splitk"),
    ((33, 17, 129), "tbmm:splitk"),     # the last chunk shares 127 elements with the first
    ((20, 100, 1003), "tbmm:splitk"),
    ((130, 70, 254), "tbmm:splitk"),
    ((1101, 1000, 33), "tbmm:tile"),    # the last chunk of 32 shares 31 elements with the first
    ((1100, 1001, 67), "tbmm:tile"),
    ((1500, 1500, 66), "tbmm:wave"),
    # short reductions, or little more than whole chunks: with enough tiles the wave-level kernel, by its estimate
    ((601, 203, 7), "tbmm:wave"),       # odd rows: loads of one element
    ((115, 1632, 148), "tbmm:wave"),    # of four
    ((1219, 411, 134), "tbmm:wave"),   # of two
    ((650, 456, 144), "tbmm:splitk"),
    ((601, 79, 7), "tbmm:splitk"),      # a narrow result would be a wavefront per 16 rows
    ((1005, 1050, 21), "tbmm:wave"),    # several tiles per wavefront
    ((1012, 1571, 43), "tbmm:tile"),
]


@pytest.mark.parametrize("shape,path", PRODUCTS)
def test_product(shape, path, oracle_threads):
    from paper_1802_04730_amd import tc355 as tc
    N, M, K = shape
    X, Y = inputs.make_tbmm(1, N, M, K, seed=N + M + K)
    buf, Z = guarded((1, N, M))
    tc.tc_tbmm(dev(X), dev(Y), Z)
    torch.cuda.synchronize()
    assert tc.last_path() == path
    err = parity_error(Z.cpu().numpy().astype(np.float64), oracle.tbmm(X, Y))
    print("product %s: parity error %.3e" % (shape, err), flush=True)
    assert err <= TIGHT and clean(buf)


@pytest.mark.parametrize("shape", [(17, 33, 7), (33, 17, 129), (1101, 1000, 33)])
def test_product_keeps_infinities_where_they_are(shape, oracle_threads):
    """Elements that two pieces or chunks share count once, and as zero in both operands elsewhere."""
    from paper_1802_04730_amd import tc355 as tc
    N, M, K = shape
    X, Y = (np.abs(a) + 0.1 for a in inputs.make_tbmm(1, N, M, K, seed=9))
    for k in (0, K // 2, K - 2, K - 1):
        X[0, k % N, k] = np.inf
    X, Y = X.astype(np.float32), Y.astype(np.float32)
    ref = oracle.tbmm(X, Y)
    buf, Z = guarded((1, N, M))
    tc.tc_tbmm(dev(X), dev(Y), Z)
    got = Z.cpu().numpy()
    assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and not np.isnan(got).any()


# batch, widths
CHAINS = [
    (1, (7, 5, 3)),
    (19, (41, 50, 67, 16, 24)),
    (300, (429, 1000, 600, 250)),
    (130, (129, 131, 5, 259)),
    (2000, (33, 301, 65)),              # 64 x 64 blocks, then tiles on fp64 activations
    (65, (3, 66, 130, 2)),              # a reduction of 3 on the wave-level kernel, then pieces moved back in fp64
]


@pytest.mark.parametrize("batch,dims", CHAINS)
@pytest.mark.parametrize("keep", [True, False])
def test_chain_of_any_widths(batch, dims, keep, oracle_threads):
    from paper_1802_04730_amd import tc355 as tc
    n = len(dims) - 1
    I, Ws, bs = inputs.make_mlp(batch, dims, seed=batch, w_std=0.1)
    ref = oracle.mlp_fcrelu(I, Ws, bs)
    outs = [guarded((batch, d)) for d in dims[1:]]
    O = [o[1] if keep or l == n - 1 else None for l, o in enumerate(outs)]
    ws = torch.full((tc.tc_mlp_fcrelu_workspace_bytes(batch, dims),), 0xCD, dtype=torch.uint8, device="cuda")
    tc.tc_mlp_fcrelu(dev(I), [dev(w) for w in Ws], [dev(b) for b in bs], O, ws)
    torch.cuda.synchronize()
    for l in range(n):
        assert clean(outs[l][0])
        if O[l] is not None:
            err = parity_error(O[l].cpu().numpy().astype(np.float64), ref[l])
            assert err <= TIGHT, (l, err)
    assert int(ws[:256].view(torch.int32)[33]) == 0  # no wait gave up: there are none
