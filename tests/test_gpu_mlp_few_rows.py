"""Chains of fewer than 16 rows: one launch per layer by default, the row kernel (whose only tile of rows is then partly empty)
where the caller asks for it.  Both against the float64 oracle to one fp32 rounding, with guarded outputs and the error word."""
import numpy as np
import pytest
import torch

import oracle
from paper_1802_04730_amd import inputs
from paper_1802_04730_amd.metric import parity_error

pytestmark = pytest.mark.gpu

TIGHT = 2.5e-7
GUARD = 64


@pytest.mark.parametrize("kernel", ["per_layer", "rows"])
@pytest.mark.parametrize("batch,dims", [(1, (1024, 1024, 512, 256)), (2, (128, 256, 1024, 128)), (5, (256, 1024, 200)), (15, (1024, 1000))])
def test_few_rows(batch, dims, kernel, oracle_threads):
    from paper_1802_04730_amd import tc355 as tc
    I, Ws, bs = inputs.make_mlp(batch, dims, seed=batch, w_std=0.05)
    ref = oracle.mlp_fcrelu(I, Ws, bs)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    bufs = [torch.full((batch * d + 2 * GUARD,), 777.0, device="cuda") for d in dims[1:]]
    O = [b[GUARD:GUARD + batch * d].view(batch, d) for b, d in zip(bufs, dims[1:])]
    nbytes = tc.tc_mlp_fcrelu_workspace_bytes(batch, dims)
    ws = torch.full((nbytes,), 0xAB, dtype=torch.uint8, device="cuda") if nbytes else None
    with tc.option(tc.TC_OPT_MLP_KERNEL, tc.TC_MLP_ROWS if kernel == "rows" else tc.TC_MLP_AUTO):
        tc.tc_mlp_fcrelu(dev(I), [dev(w) for w in Ws], [dev(b) for b in bs], O, ws)
        assert tc.last_path() == "mlp:" + kernel
    torch.cuda.synchronize()
    if nbytes:
        assert int(ws[:256].view(torch.int32)[33]) == 0
    for l, (b, o) in enumerate(zip(bufs, O)):
        err = parity_error(o.cpu().numpy().astype(np.float64), ref[l])
        print("mlp %d x %s on %s, layer %d: parity error %.3e" % (batch, dims, kernel, l, err), flush=True)
        assert err <= TIGHT
        assert bool((b[:GUARD] == 777.0).all()) and bool((b[GUARD + o.numel():] == 777.0).all())
