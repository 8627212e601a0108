"""GPU parity of the shape-generic grouped convolution (16- and 4-filter MFMA tiles over one LDS band) against the
float64 oracle: one fp32 rounding of the exact result (2.5e-7 on the metric, as for every fp64 kernel)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1802_04730_amd import inputs
from paper_1802_04730_amd.metric import parity_error

pytestmark = pytest.mark.gpu

TIGHT = 2.5e-7
GUARD = 64

# (N, G, C, F, H, W, KH, KW)
SHAPES = [
    (2, 2, 5, 3, 9, 11, 3, 3),        # one quad, the last filter missing; 45 taps: the last step has one
    (1, 3, 6, 8, 13, 17, 3, 2),       # two quads; 36 taps in W1's order
    (3, 2, 8, 12, 20, 19, 3, 3),      # three quads; channels in fours
    (2, 2, 12, 16, 33, 45, 3, 3),     # one tile of 16 (84 pixel tiles: shares of 3 and 4)
    (2, 3, 12, 20, 33, 45, 3, 3),     # a tile and a quad
    (1, 2, 9, 22, 31, 30, 3, 3),      # a tile and two quads, two filters missing
    (1, 2, 7, 27, 14, 14, 5, 5),      # a tile and three quads
    (2, 1, 13, 32, 21, 23, 3, 3),     # two tiles
    (2, 2, 40, 40, 12, 14, 3, 3),     # two blocks of 20 filters
    (1, 2, 70, 33, 11, 12, 5, 5),     # 1750 taps: chunks of channels; two blocks, the second short
    (1, 1, 37, 21, 40, 64, 5, 5),     # chunks whose last one is no multiple of four channels
    (11, 3, 6, 10, 7, 7, 3, 3),       # several images per job, the last job with fewer
    (5, 2, 3, 5, 4, 5, 3, 3),         # 6 pixels per image
    (3, 40, 4, 4, 14, 14, 3, 3),      # many groups: runs that cross group boundaries
    (9, 25, 11, 18, 16, 21, 1, 1),    # 1 x 1 filters
    (2, 5, 4, 7, 1, 64, 1, 5),        # a single row
    (2, 3, 10, 6, 64, 3, 3, 3),       # one output column
    # two images of 6 channels behind one of 12, and the like (tests/test_gconv_mix_plan.py): several images per job and
    # several chunks, in runs of more than one job
    (33, 63, 42, 2, 9, 17, 3, 3),
    (62, 54, 30, 3, 18, 6, 3, 3),
]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("with_bias", [True, False])
def test_gconv_generic(shape, with_bias, oracle_threads):
    from paper_1802_04730_amd import tc355 as tc
    N, G, C, F, H, W, KH, KW = shape
    I, W1, bias = inputs.make_gconv(*shape, seed=C + F)
    ref = oracle.group_conv(I, W1, bias if with_bias else None)
    buf = torch.full((ref.size + 2 * GUARD,), 777.0, device="cuda")
    O = buf[GUARD:GUARD + ref.size].view(ref.shape)
    dev = lambda a: torch.from_numpy(a).cuda()
    tc.tc_group_conv(dev(I), dev(W1), dev(bias) if with_bias else None, O)
    torch.cuda.synchronize()
    assert tc.last_path() == "gconv:mix"
    err = parity_error(O.cpu().numpy().astype(np.float64), ref)
    print("gconv generic %s: parity error %.3e" % (shape, err), flush=True)
    assert err <= TIGHT
    assert bool((buf[:GUARD] == 777.0).all()) and bool((buf[GUARD + ref.size:] == 777.0).all())


def test_gconv_generic_keeps_infinities_out_of_the_padding(oracle_threads):
    """Unused k slots of a last step (27 taps: one) multiply nothing: an Inf gives Inf where the definition does and leaves
    every output that does not read it finite."""
    from paper_1802_04730_amd import tc355 as tc
    I, W1, bias = inputs.make_gconv(2, 2, 3, 6, 12, 13, 3, 3, seed=5)
    W1 = np.abs(W1) + 0.01
    I[1, 0, 2, 11, 12] = np.inf
    I[0, 1, 0, 0, 0] = np.inf
    ref = oracle.group_conv(I, W1, bias)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    O = torch.full(ref.shape, float("nan"), device="cuda")
    tc.tc_group_conv(dev(I), dev(W1), dev(bias), O)
    got = O.cpu().numpy()
    assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and np.isposinf(ref).sum() == 12
    assert not np.isnan(got).any()


@pytest.mark.parametrize("shape,path", [
    ((16, 32, 16, 16, 22, 22, 3, 3), "gconv:lds"),   # one block of 448 pixels per image, enough of them
    ((4, 33, 16, 16, 30, 30, 3, 3), "gconv:lds"),    # two
    ((3, 32, 16, 16, 30, 30, 3, 3), "gconv:mix"),    # too few of them
    ((8, 32, 16, 16, 21, 22, 3, 3), "gconv:mix"),    # 380 pixels leave the block 15 % empty
    ((4, 31, 4, 4, 56, 56, 3, 3), "gconv:mix"),      # few (image, group) pairs: pieces of an image
    ((8, 31, 4, 4, 56, 56, 3, 3), "gconv:quad"),     # one workgroup for each
    ((2, 31, 8, 8, 28, 28, 3, 3), "gconv:mix"),
    ((4, 31, 8, 8, 28, 28, 3, 3), "gconv:quad"),
    # the 4x4x4-block kernel with a workgroup for each (image, group): last bands of fewer rows, odd heights, a short image,
    # 8-byte staging loads at widths 58 and 30
    ((9, 29, 4, 4, 53, 56, 3, 3), "gconv:quad"),
    ((16, 16, 4, 4, 5, 56, 3, 3), "gconv:quad"),
    ((8, 32, 4, 4, 58, 58, 3, 3), "gconv:quad"),
    ((16, 17, 4, 4, 21, 58, 3, 3), "gconv:quad"),
    ((9, 29, 8, 8, 31, 28, 3, 3), "gconv:quad"),
    ((8, 32, 8, 8, 30, 30, 3, 3), "gconv:quad"),
    ((16, 17, 8, 8, 17, 30, 3, 3), "gconv:quad"),
    ((8, 31, 4, 4, 21, 58, 3, 3), "gconv:quad"),     # few rows: one workgroup's two bands are done before the pieces are
    ((3, 31, 4, 4, 58, 58, 3, 3), "gconv:mix"),
    ((4, 31, 8, 8, 17, 30, 3, 3), "gconv:mix"),
    # too little to stage: the wave-level kernel, in strips of 4, 2 and 1 tiles of 16 pixels
    ((2, 3, 4, 19, 9, 10, 1, 1), "gconv:wave"),
    ((2, 3, 4, 5, 6, 7, 1, 1), "gconv:wave"),
    ((1, 2, 2, 3, 5, 6, 3, 2), "gconv:wave"),
    ((5, 2, 2, 17, 3, 4, 1, 2), "gconv:wave"),
    # one group of at least 64 filters: the strided convolution's kernels
    ((2, 1, 12, 70, 15, 17, 3, 3), "gconv:split"),
    ((9, 1, 9, 70, 38, 39, 3, 3), "gconv:tile"),
])
def test_gconv_both_sides_of_the_dispatch(shape, path, oracle_threads):
    from paper_1802_04730_amd import tc355 as tc
    I, W1, bias = inputs.make_gconv(*shape, seed=shape[0] + shape[4])
    ref = oracle.group_conv(I, W1, bias)
    dev = lambda a: torch.from_numpy(a).cuda()
    O = torch.full(ref.shape, float("nan"), device="cuda")
    tc.tc_group_conv(dev(I), dev(W1), dev(bias), O)
    torch.cuda.synchronize()
    assert tc.last_path() == path
    assert parity_error(O.cpu().numpy().astype(np.float64), ref) <= TIGHT
