"""What the int8 kernels with a scale per row and block promise of an operand: off by at most 2^-32 of its block's largest magnitude.
Rows that hold 1 and, else, 2^-31: the ones meet zeros (or cancel), so that the outputs are what became of the small elements.  A
scale that fills one bit less than the digits have turns every one of them into 0."""
import numpy as np
import pytest
import torch

from paper_1802_04730_amd.metric import parity_error

pytestmark = pytest.mark.gpu

SMALL = 2.0 ** -31


@pytest.mark.parametrize("M,K,workspace", [(8192, 256, False), (8192, 2048, True)])
def test_small_elements_of_a_row(M, K, workspace):
    from paper_1802_04730_amd import tc355 as tc
    X, Y = torch.full((1, 128, K), SMALL), torch.ones(1, M, K)
    X[:, :, ::128], Y[:, :, ::128] = 1.0, 0.0
    Z = torch.full((1, 128, M), float("nan"), device="cuda")
    if workspace:
        ws = torch.empty(tc.tc_tbmm_workspace_bytes(1, 128, M, K), dtype=torch.uint8, device="cuda")
        tc.tc_tbmm_ws(X.cuda(), Y.cuda(), Z, ws)
        assert tc.last_path() == "tbmm:i8_presliced"
    else:
        tc.tc_tbmm(X.cuda(), Y.cuda(), Z)
        assert tc.last_path() == "tbmm:i8"
    terms = K - K // 128
    # every term off by 2^-32 * 1, a fortieth of that for dropped digit products
    assert float((Z.cpu().double() - terms * SMALL).abs().max()) <= terms * 2.0 ** -32 * 1.025


def test_small_elements_of_a_filter():
    from paper_1802_04730_amd import tc355 as tc
    N, C, F, H, W = 2, 32, 128, 10, 10
    Wt = torch.full((F, C * 9), SMALL)
    Wt[:, ::64] = 1.0
    Wt[:, 64::128] = -1.0  # one of each sign in the blocks of 128, but the last one: 1 alone
    Wt[:, 256] = SMALL
    I, O = torch.ones(N, C, H, W), torch.full((N, F, H - 2, W - 2), float("nan"), device="cuda")
    tc.tc_sconv2d(I.cuda(), Wt.reshape(F, C, 3, 3).cuda(), None, O, 1, 1)
    assert tc.last_path() == "sconv:i8"
    terms = C * 9 - 4
    assert float((O.cpu().double() - terms * SMALL).abs().max()) <= terms * 2.0 ** -32 * 1.025


def test_heavy_tailed_rows():
    """Log-normal magnitudes, sigma 2, on both operands: below 2e-6 on the metric, as the header says."""
    from paper_1802_04730_amd import tc355 as tc
    for seed in (0, 3, 4, 5):
        rng = np.random.default_rng(seed)
        X = (rng.standard_normal((128, 1024)) * np.exp(rng.normal(size=(128, 1024)) * 2.0)).astype(np.float32)
        Y = (rng.standard_normal((96, 1024)) * np.exp(rng.normal(size=(96, 1024)) * 2.0)).astype(np.float32)
        Yall = np.zeros((8192, 1024), dtype=np.float32)
        Yall[:96] = Y
        Z = torch.full((1, 128, 8192), float("nan"), device="cuda")
        tc.tc_tbmm(torch.from_numpy(X[None]).cuda(), torch.from_numpy(Yall[None]).cuda(), Z)
        assert tc.last_path() == "tbmm:i8"
        err = parity_error(Z[0, :, :96].cpu().numpy().astype(np.float64), X.astype(np.float64) @ Y.T.astype(np.float64))
        print("tmm, log-normal of sigma 2, seed %d: parity error %.3e" % (seed, err), flush=True)
        assert err <= 2e-6
