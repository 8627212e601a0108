"""GPU parity of convolutions with few blocks of 64 filters (split reduction) against the float64 oracle: one fp32 rounding
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

# (N, C, F, H, W, KH, KW, sh, sw)
SHAPES = [
    (1, 1, 1, 1, 1, 1, 1, 1, 1),          # one tap, one output
    (1, 21, 64, 46, 46, 7, 7, 2, 2),      # 1029 taps: sixteen chunks and 5 taps
    (1, 7, 33, 17, 18, 3, 3, 1, 1),       # 63 taps: one short chunk; the third filter tile has one
    (2, 16, 17, 9, 11, 2, 2, 1, 2),       # 64 taps: one whole chunk
    (3, 13, 16, 12, 10, 5, 1, 1, 3),      # 65 taps: one more; pixels of several images in a tile
    (1, 129, 20, 9, 9, 1, 1, 1, 1),       # 1 x 1 filters, two chunks and one tap
    (2, 193, 215, 19, 21, 4, 4, 1, 1),    # many filters and taps: blocks of 32 filters
    (1, 1500, 36, 8, 9, 3, 3, 2, 2),      # 13500 taps: the table of tap offsets takes a third of the LDS
]

# enough blocks of 64 filters for the kernel without a split (sconv_tile.hpp)
TILE_SHAPES = [
    (15, 3, 70, 33, 36, 3, 3, 1, 1),      # 27 taps: one chunk and 11; 15810 pixels; the second filter block has 6
    (9, 7, 129, 27, 24, 3, 3, 1, 1),      # 63 taps; three filter blocks, the last one a single filter
    (13, 13, 65, 25, 55, 5, 1, 1, 2),     # 65 taps, strides 1 and 2
    (1, 64, 100, 110, 110, 3, 3, 1, 1),   # 576 taps in fours, two blocks
    (3, 5, 256, 112, 109, 2, 2, 1, 1),    # 20 taps, blocks of 64 pixels
    (1, 174, 256, 35, 69, 1, 1, 1, 1),    # both estimated alike
    (9, 163, 155, 35, 47, 1, 1, 2, 2),    # strides that step over the filters
]


@pytest.mark.parametrize("shape,path", [(s, "sconv:split") for s in SHAPES] + [(s, "sconv:tile") for s in TILE_SHAPES])
@pytest.mark.parametrize("with_bias", [True, False])
def test_sconv_split(shape, path, with_bias, oracle_threads):
    from paper_1802_04730_amd import tc355 as tc
    N, C, F, H, W, KH, KW, sh, sw = shape
    I, Wt, bias = inputs.make_sconv2d(N, C, F, H, W, KH, KW, seed=C + F)
    ref = oracle.sconv2d(I, Wt, bias if with_bias else None, sh, sw)
    buf = torch.full((ref.size + 2 * GUARD,), 777.0, device="cuda")
    O = buf[GUARD:GUARD + ref.size].view(ref.shape)
    dev = lambda a: torch.from_numpy(a).cuda()
    tc.tc_sconv2d(dev(I), dev(Wt), dev(bias) if with_bias else None, O, sh, sw)
    torch.cuda.synchronize()
    assert tc.last_path() == path
    err = parity_error(O.cpu().numpy().astype(np.float64), ref)
    print("sconv %s: parity error %.3e" % (shape, err), flush=True)
    assert err <= TIGHT
    assert bool((buf[:GUARD] == 777.0).all()) and bool((buf[GUARD + ref.size:] == 777.0).all())


def test_sconv_split_keeps_infinities_out_of_the_padding(oracle_threads):
    """Taps past the end read some element of the input and count as zeros: an Inf reaches its own outputs only."""
    from paper_1802_04730_amd import tc355 as tc
    I, Wt, bias = inputs.make_sconv2d(1, 7, 20, 11, 12, 3, 3, seed=8)
    Wt = np.abs(Wt) + np.float32(0.01)
    I[0, 0, 0, 0] = np.inf
    I[0, 6, 10, 11] = np.inf
    ref = oracle.sconv2d(I, Wt, bias, 1, 1)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    O = torch.full(ref.shape, float("nan"), device="cuda")
    tc.tc_sconv2d(dev(I), dev(Wt), dev(bias), O, 1, 1)
    got = O.cpu().numpy()
    assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and np.isposinf(ref).sum() == 40
    assert not np.isnan(got).any()
