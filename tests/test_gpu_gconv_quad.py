"""GPU parity of the grouped convolution with 4 or 8 channels per group in bands of an image, at the edges of the bands and of the
pairs that share an XCD, against the float64 oracle: one fp32 rounding of the exact result (2.5e-7 on the metric, as for every
fp64 kernel)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1802_04730_amd import inputs
from paper_1802_04730_amd.metric import parity_error

pytestmark = pytest.mark.gpu

TIGHT = 2.5e-7
GUARD = 64

# (N, G, channels and filters, H, W): at least 125 pairs; output rows per band 9, 8, 13, 14 at widths 56, 58, 28, 30
SHAPES = [
    (5, 25, 4, 11, 56),    # one whole band; 125 pairs: three of the last eight are not there
    (5, 25, 4, 12, 56),    # one row in the second band
    (32, 4, 4, 3, 56),     # a single output row
    (7, 19, 4, 10, 58),    # one whole band
    (7, 19, 4, 27, 58),    # three and one row
    (43, 3, 8, 15, 28),    # one whole band
    (43, 3, 8, 28, 28),    # two
    (129, 1, 8, 29, 28),   # ... and one row; one group
    (1, 131, 8, 16, 30),   # one whole band of one image
    (1, 131, 8, 30, 30),   # two
    (2, 70, 8, 31, 30),    # ... and one row
]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("bias", [True, False])
def test_bands(shape, bias, oracle_threads):
    from paper_1802_04730_amd import tc355 as tc
    N, G, C, H, W = shape
    I, W1, b = inputs.make_gconv(N, G, C, C, H, W, 3, 3, seed=sum(shape))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    size = N * G * C * (H - 2) * (W - 2)
    buf = torch.full((size + 2 * GUARD,), 777.0, device="cuda")
    O = buf[GUARD:GUARD + size].view(N, G, C, H - 2, W - 2)
    tc.tc_group_conv(dev(I), dev(W1), dev(b) if bias else None, O)
    torch.cuda.synchronize()
    assert tc.last_path() == "gconv:quad"
    assert bool((buf[:GUARD] == 777.0).all()) and bool((buf[GUARD + size:] == 777.0).all())
    err = parity_error(O.cpu().numpy().astype(np.float64), oracle.group_conv(I, W1, b if bias else None))
    print("gconv %s: parity error %.3e" % (shape, err), flush=True)
    assert err <= TIGHT
