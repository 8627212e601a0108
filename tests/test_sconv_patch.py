"""Strided convolution on int8 with the input sliced where it lies (csrc/sconv_patch.hpp): which layers take it (the function that
the library asks, in csrc/sconv_patch_plan.hpp, compiled by the system's C++ compiler, for 256 compute units or as many as the
device has) and, on the GPU, parity with the float64 oracle.  4e-6 on the metric and a quarter of the bar on heavy-tailed operands are what every int8 kernel is held to."""
import ctypes
import os
import subprocess

import numpy as np
import pytest
import torch

import oracle
from paper_1802_04730_amd import inputs
from paper_1802_04730_amd.metric import PARITY_BAR, parity_error

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TIGHT_I8 = 4e-6

# (N, C, F, H, W, KH, KW, sh, sw): filters per workgroup, pixel tiles per wavefront
LAYERS = {
    (13, 32, 32, 184, 9, 3, 3, 1, 1): (32, 2),   # an only stage
    (27, 32, 96, 27, 33, 3, 3, 2, 1): (32, 3),   # strides that differ
    (12, 96, 96, 45, 46, 3, 3, 1, 1): (32, 5),   # three stages; runs that start and end inside rows
    (28, 32, 160, 52, 9, 3, 3, 1, 1): (32, 6),
    (1, 32, 320, 166, 12, 3, 3, 1, 1): (64, 2),
    (11, 32, 448, 68, 14, 9, 1, 2, 2): (64, 3),  # nine taps in a column
    (9, 64, 64, 58, 57, 3, 3, 1, 1): (64, 4),    # two stages
    (29, 32, 192, 14, 49, 3, 3, 2, 1): (64, 5),
    (15, 32, 384, 28, 30, 3, 3, 2, 2): (128, 3),
    (8, 64, 128, 61, 56, 3, 3, 2, 1): (128, 4),
    (19, 32, 128, 62, 47, 9, 1, 2, 2): (128, 5),
    (32, 64, 128, 56, 56, 3, 3, 2, 2): (128, 6),
}


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("sconv_patch")
    (d / "plan.cpp").write_text('#include "sconv_patch_plan.hpp"\n'
                                'extern "C" int plan(const int64_t* a, int64_t G, int cus, int64_t* o) {\n'
                                '  tc355::SconvPatchPlan p{};\n  tc355::SconvI8Deal d{};\n'
                                '  if (!tc355::plan_sconv_patch(a[0], G, a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], cus, &p)) return 0;\n'
                                '  const int64_t OH = (a[3] - a[5]) / a[7] + 1, OW = (a[4] - a[6]) / a[8] + 1;\n'
                                '  if (!tc355::deal_sconv_i8(a[0] * OH * OW, a[2], a[1] * a[5] * a[6], G, cus, &d)) return 0;\n'
                                '  o[0] = p.tf; o[1] = p.tiles; o[2] = p.px; o[3] = p.blocks;\n'
                                '  return tc355::sconv_by_patches(d, a[0], G, a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], cus, &p) ? 2 : 1;\n}\n'
                                'extern "C" unsigned magic(int d) { return tc355::sp_magic(d); }\n')
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_1802_04730_amd", "csrc"),
                    "-o", str(d / "plan.so"), str(d / "plan.cpp")], check=True)
    lib = ctypes.CDLL(str(d / "plan.so"))

    def ask(layer, G=1, cus=256):
        o = (ctypes.c_int64 * 4)()
        return lib.plan((ctypes.c_int64 * 9)(*layer), ctypes.c_int64(G), ctypes.c_int(cus), o), tuple(o)

    ask.magic = lib.magic
    return ask


def test_layers_take_the_kernel(plan):
    for layer, said in LAYERS.items():
        took, (tf, tiles, px, blocks) = plan(layer)
        assert took == 2 and (tf, tiles) == said, (layer, took, tf, tiles)


def test_what_the_kernel_takes_for_granted(plan):
    rng = np.random.default_rng(3)
    seen = 0
    for _ in range(4000):
        KH, KW = ((3, 3), (1, 9), (9, 1))[rng.integers(0, 3)]
        H, W = int(rng.integers(KH, 300)), int(rng.integers(KW, 300))
        sh, sw = int(rng.integers(1, 5)), int(rng.integers(1, 5))
        layer = (int(rng.integers(1, 40)), 32 * int(rng.integers(1, 9)), 32 * int(rng.integers(1, 13)), H, W, KH, KW, sh, sw)
        took, (tf, tiles, px, blocks) = plan(layer, int(rng.integers(1, 9)))
        if not took:
            continue
        seen += 1
        OH, OW = (H - KH) // sh + 1, (W - KW) // sw + 1
        assert layer[2] % tf == 0 and 1 <= tiles <= 6 and px <= 16 * tiles * (128 // tf)
        assert blocks * px >= OH * OW > (blocks - 1) * px
        for b in range(blocks):
            p0, n = b * px, min(px, OH * OW - b * px)
            rows = ((p0 + n - 1) // OW - p0 // OW) * sh + KH  # input rows under the run
            assert 4 <= rows * W <= 640
            assert p0 % OW + n <= 2048  # what a division by multiplication gets
    assert seen > 1000
    n = np.arange(2048, dtype=np.int64)
    for d in range(1, 641):
        m = plan.magic(d)
        assert (n * m < 1 << 32).all() and np.array_equal((n * m) >> 21, n // d), d


@pytest.fixture
def run(plan):
    """A call that this device does by patches.  (tc355_last_path names the int8 convolutions alike: that the library's own choice says
    so is what tells this one from the other.)"""
    cus = torch.cuda.get_device_properties(0).multi_processor_count

    def call(I, Wt, bias, sh, sw, shape, groups=None):
        N, C, H, W = (I.shape[0],) + I.shape[-3:]
        assert plan((N, C, shape[-3], H, W) + Wt.shape[-2:] + (sh, sw), groups or 1, cus)[0] == 2
        return launch(I, Wt, bias, sh, sw, shape, groups)

    return call


def launch(I, Wt, bias, sh, sw, shape, groups):
    from paper_1802_04730_amd import tc355 as tc
    dev = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    n = int(np.prod(shape))
    buf = torch.full((n + 512,), 7.0, device="cuda")
    O = buf[256:256 + n].view(shape)
    if groups is None:
        tc.tc_sconv2d(dev(I), dev(Wt), dev(bias), O, sh, sw)
        assert tc.last_path() == "sconv:i8"
    else:
        tc.tc_group_conv(dev(I), dev(Wt), dev(bias), O)
        assert tc.last_path() == "gconv:i8_taps"
    torch.cuda.synchronize()
    assert torch.all(buf[:256] == 7.0) and torch.all(buf[256 + n:] == 7.0)
    return O.cpu().numpy().astype(np.float64)


@pytest.mark.gpu
@pytest.mark.parametrize("layer", list(LAYERS))
def test_parity(run, layer, oracle_threads):
    N, C, F, H, W, KH, KW, sh, sw = layer
    I, Wt, bias = inputs.make_sconv2d(N, C, F, H, W, KH, KW, seed=inputs.SEED_BASE + 300 + C)
    bias = bias if C != 64 else None
    ref = oracle.sconv2d(I, Wt, bias, sh, sw)
    err = parity_error(run(I, Wt, bias, sh, sw, ref.shape), ref)
    print("sconv2d by patches %s: parity error %.3e" % (layer, err), flush=True)
    assert err <= TIGHT_I8


GROUPED = (20, 4, 32, 32, 33, 34, 3, 3)  # N, G, C, F, H, W, KH, KW


def test_grouped_layer_takes_the_kernel(plan):
    N, G, C, F, H, W, KH, KW = GROUPED
    assert plan((N, C, F, H, W, KH, KW, 1, 1), G)[0] == 2


@pytest.mark.gpu
def test_groups(run, oracle_threads):
    N, G, C, F, H, W, KH, KW = GROUPED
    I, W1, bias = inputs.make_gconv(N, G, C, F, H, W, KH, KW, seed=inputs.SEED_BASE + 310)
    ref = oracle.group_conv(I, W1, bias)
    assert parity_error(run(I, W1, bias, 1, 1, ref.shape, G), ref) <= TIGHT_I8
    I[3, 2, :, :, W // 2:] *= np.float32(1e-5)  # runs of one group of one image to do by taps
    ref = oracle.group_conv(I, W1, None)
    got = run(I, W1, None, 1, 1, ref.shape, G)
    for g in range(G):
        allowed = own_bound(I[:4, g], W1[g], 1, 1) + np.abs(ref[:4, g]) * 2.0 ** -24
        assert (np.abs(got[:4, g] - ref[:4, g]) <= allowed).all()


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["lognormal", "student3", "sparse", "tiny"])
def test_heavy_tailed_operands(run, kind, oracle_threads):
    N, C, F, H, W, KH, KW, sh, sw = (9, 64, 64, 58, 57, 3, 3, 1, 1)
    I, Wt, bias = inputs.make_sconv2d(N, C, F, H, W, KH, KW, seed=77)
    rng = np.random.default_rng(9)
    mag = {"lognormal": lambda a: np.exp(rng.normal(size=a.shape) * 1.5), "student3": lambda a: np.abs(rng.standard_t(3, size=a.shape)),
           "sparse": lambda a: np.where(rng.random(a.shape) < 0.01, 300.0, 1.0),
           # denormal inputs.  (Filters of 2^40 lift the outputs to 2^-90: where outputs are denormal as well, a rounding is half of
           # 2^-149, 2^-10 of an output of 2^-140, whatever computes it.)
           "tiny": lambda a: np.full(a.shape, 2.0 ** -130 if a is I else 2.0 ** 40)}[kind]
    I, Wt = (I * mag(I)).astype(np.float32), (Wt * mag(Wt)).astype(np.float32)
    bias = bias if kind != "tiny" else None
    ref = oracle.sconv2d(I, Wt, bias, sh, sw)
    err = parity_error(run(I, Wt, bias, sh, sw, ref.shape), ref)
    print("sconv2d by patches, %s: parity error %.3e" % (kind, err), flush=True)
    assert err <= PARITY_BAR / 4


@pytest.mark.gpu
def test_nan_and_inf_stay_in_the_outputs_that_read_them(run, oracle_threads):
    N, C, F, H, W, KH, KW, sh, sw = (32, 64, 128, 56, 56, 3, 3, 2, 2)
    I, Wt, bias = inputs.make_sconv2d(N, C, F, H, W, KH, KW, seed=81)
    ref = oracle.sconv2d(I, Wt, bias, sh, sw)
    In = I.copy()
    In[1, 5, 6, 8] = np.nan    # rows 6 = 2*2 + 2 = 2*3 + 0, columns 8 = 2*3 + 2 = 2*4 + 0; first stage
    In[7, 63, 55, 55] = np.inf  # under no window
    In[7, 40, 54, 54] = -np.inf  # row and column 54 = 2*26 + 2 alone; second stage
    got = run(In, Wt, bias, sh, sw, ref.shape)
    hit = np.zeros(ref.shape, dtype=bool)
    hit[1, :, 2:4, 3:5] = True
    hit[7, :, 26, 26] = True
    assert np.isnan(got[hit]).all() and not np.isnan(got[~hit]).any()
    assert parity_error(np.where(hit, ref, got), ref) <= TIGHT_I8
    # the same in runs that are done by taps: the NaN in the stage that finds it out, the other Inf in the one before
    hit[7, :, 26, 26] = False
    In[7, 40, 54, 54] = I[7, 40, 54, 54]
    In[1, 9, 0, 55] = In[7, 63, 0, 0] = 1e6
    In[7, 20, 10, 10] = np.inf
    hit[7, :, 4:6, 4:6] = True
    ref1 = ref.copy()
    ref1[[1, 7]] = oracle.sconv2d(np.where(np.isfinite(In[[1, 7]]), In[[1, 7]], 0), Wt, bias, sh, sw)
    got = run(In, Wt, bias, sh, sw, ref.shape)
    assert np.isnan(got[hit]).all() and not np.isnan(got[~hit]).any()
    hit[7, :, 0, 0] = True  # (reads 1e6 itself)
    assert parity_error(np.where(hit, ref, got), np.where(hit, ref, ref1)) <= TIGHT_I8
    Wn = Wt.copy()
    Wn[77, 3, 1, 2] = np.nan
    Wn[5, 60, 2, 2] = np.inf
    got = run(I, Wn, bias, sh, sw, ref.shape)
    hit = np.zeros(ref.shape, dtype=bool)
    hit[:, [5, 77]] = True
    assert np.isnan(got[hit]).all() and not np.isnan(got[~hit]).any()
    assert parity_error(np.where(hit, ref, got), ref) <= TIGHT_I8


@pytest.mark.gpu
@pytest.mark.parametrize("layer,channel,at", [
    ((32, 64, 128, 56, 56, 3, 3, 2, 2), 19, (7, 9)),   # the second 16 channels of a stage start 16 bytes later at even strides
    ((32, 64, 128, 56, 56, 3, 3, 2, 2), 48, (55, 1)),  # under no window (rows 0 .. 54)
    ((9, 64, 64, 58, 57, 3, 3, 1, 1), 31, (57, 56)),
    ((9, 64, 64, 58, 57, 3, 3, 1, 1), 60, (20, 0)),
])
def test_inf_in_the_second_half_of_a_stage(run, layer, channel, at, oracle_threads):
    N, C, F, H, W, KH, KW, sh, sw = layer
    I, Wt, bias = inputs.make_sconv2d(N, C, F, H, W, KH, KW, seed=83)
    ref = oracle.sconv2d(I, Wt, bias, sh, sw)
    I[2, channel, at[0], at[1]] = np.inf
    got = run(I, Wt, bias, sh, sw, ref.shape)
    hit = np.zeros(ref.shape, dtype=bool)
    for oh in range(ref.shape[2]):
        for ow in range(ref.shape[3]):
            if oh * sh <= at[0] < oh * sh + KH and ow * sw <= at[1] < ow * sw + KW:
                hit[2, :, oh, ow] = True
    assert np.isnan(got[hit]).all() and not np.isnan(got[~hit]).any()
    assert parity_error(np.where(hit, ref, got), ref) <= TIGHT_I8


def own_bound(I, Wt, sh, sw):
    """What one scale per 128 taps of the output's OWN pixel and filter could do to it: K * 2^-30.5 * the two largest magnitudes, block by
    block.  (By patches the worst case is K * 2^-27.8 with blocks of 16 channels, where every rounding has the same sign and a window just
    passes; sums of rounding errors of either sign are far from it.)"""
    N, F, K = I.shape[0], Wt.shape[0], Wt[0].size
    taps = torch.nn.functional.unfold(torch.from_numpy(I).double().abs(), Wt.shape[2:], stride=(sh, sw)).transpose(1, 2)  # [N, pixels, K]
    filters = torch.from_numpy(Wt).double().abs().reshape(F, K)
    at = range(0, K, 128)
    tm = torch.stack([taps[:, :, a:a + 128].amax(2) for a in at], 2)
    fm = torch.stack([filters[:, a:a + 128].amax(1) * min(128, K - a) for a in at], 1)
    return (2.0 ** -30.5 * tm @ fm.T).transpose(1, 2).reshape(N, F, (I.shape[2] - Wt.shape[2]) // sh + 1, -1).numpy()


def unlike(layer, what, size, seed):
    """Operands of a layer that takes the kernel, Gaussian but for something of another size in image 1."""
    N, C, F, H, W, KH, KW, sh, sw = layer
    I, Wt, _ = inputs.make_sconv2d(N, C, F, H, W, KH, KW, seed=seed)
    if what == "a column that no window reads":
        assert (W - KW) % sw != 0
        I[1, 5, 10, W - 1] = size
    elif what == "a corner":
        I[1, C // 2 + 8, 0, 0] = size
    elif what == "a channel of zero weights":
        Wt[:, 33] = 0.0
        I[1, 33, 12, 20] = size
    elif what == "a dim region":
        I[1, :, :, W // 2:] *= size
    elif what == "dim channels":
        I[1, 16:32] *= size
    elif what == "half of a filter":
        Wt[7, :16] *= size
    return I, Wt


ODD_STRIDE, EVEN_STRIDE = (9, 64, 64, 58, 57, 3, 3, 1, 1), (32, 64, 128, 56, 56, 3, 3, 2, 2)
FLT_MAX = float(np.finfo(np.float32).max)


@pytest.mark.gpu
@pytest.mark.parametrize("layer,what,size", [
    (EVEN_STRIDE, "a column that no window reads", 1e3),
    (EVEN_STRIDE, "a column that no window reads", 1e10),
    (EVEN_STRIDE, "a corner", 1e6),
    (EVEN_STRIDE, "a channel of zero weights", -FLT_MAX),
    (EVEN_STRIDE, "a dim region", 1e-4),
    (ODD_STRIDE, "a corner", 1e3),
    (ODD_STRIDE, "a corner", -FLT_MAX),
    (ODD_STRIDE, "a channel of zero weights", 1e3),
    (ODD_STRIDE, "a channel of zero weights", 1e10),
    (ODD_STRIDE, "a dim region", 1e-6),
    (ODD_STRIDE, "a dim region", 0.2),
    (ODD_STRIDE, "a dim region", 1e-30),
    (ODD_STRIDE, "dim channels", 1e-5),
    (ODD_STRIDE, "half of a filter", 1e-5),
    (ODD_STRIDE, "half of a filter", 0.0),
    ((13, 32, 32, 184, 9, 3, 3, 1, 1), "a corner", 1e8),  # 32 filters, an only stage
    ((11, 32, 448, 68, 14, 9, 1, 2, 2), "a dim region", 1e-5),  # nine taps in a column
    ((8, 64, 256, 40, 60, 1, 9, 1, 2), "a dim region", 1e-5),  # and in a row
])
def test_elements_of_other_sizes_stay_in_the_outputs_that_read_them(run, layer, what, size, oracle_threads):
    """Every output is held to its own taps' magnitudes, whatever lies beside them in the patch."""
    N, C, F, H, W, KH, KW, sh, sw = layer
    I, Wt = unlike(layer, what, size, 91)
    OH, OW = (H - KH) // sh + 1, (W - KW) // sw + 1
    got = run(I, Wt, None, sh, sw, (N, F, OH, OW))
    images = [1, N - 1]
    ref = oracle.sconv2d(I[images], Wt, None, sh, sw)
    allowed = own_bound(I[images], Wt, sh, sw) + np.abs(ref) * 2.0 ** -24 + 2.0 ** -150
    over = np.abs(got[images] - ref) / allowed
    print("sconv2d by patches %s, %s of %g: %.3g of what is allowed" % (layer, what, size, over.max()), flush=True)
    assert over.max() <= 1.0
