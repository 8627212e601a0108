"""The binding's native calls: they make the call that the general path makes, on the stream that it uses, and leave to it
whatever they do not know to be right."""
import pytest
import torch

from paper_1802_04730_amd import inputs, tc355 as tc


def _calls(dev):
    """(name, arguments, outputs) of every entry point, small."""
    import numpy as np
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    e = lambda *s: torch.full(s, float("nan"), device=dev)
    X, Y = inputs.make_tbmm(3, 5, 7, 9, seed=1)
    Z = e(3, 5, 7)
    yield "tc_tbmm", [d(X), d(Y), Z], [Z]
    Z2 = e(3, 5, 7)
    yield "tc_tbmm_ws", [d(X), d(Y), Z2, torch.empty(64, dtype=torch.uint8, device=dev)], [Z2]
    dims = (6, 5, 4)
    I, W, b = inputs.make_mlp(3, dims, seed=2)
    O = [None, e(3, 4)]
    ws = torch.empty(tc.tc_mlp_fcrelu_workspace_bytes(3, dims), dtype=torch.uint8, device=dev)
    yield "tc_mlp_fcrelu", [d(I), [d(w) for w in W], tuple(d(x) for x in b), O, ws], [O[1]]
    I, W1, b = inputs.make_gconv(2, 3, 4, 5, 8, 9, 3, 2, seed=3)
    for bias in (b, None):
        O = e(2, 3, 5, 6, 8)
        yield "tc_group_conv", [d(I), d(W1), None if bias is None else d(bias), O], [O]
    W1, W2, X = inputs.make_kron(2, 3, 4, 5, 6, seed=4)
    Yk = e(2, 3, 5)
    yield "tc_kron", [d(W1), d(W2), d(X), Yk], [Yk]
    I, Wt, b = inputs.make_sconv2d(2, 3, 4, 9, 8, 3, 3, seed=5)
    O = e(2, 4, 4, 6)
    yield "tc_sconv2d", [d(I), d(Wt), d(b), O, 2, 1], [O]
    T = [inputs.make_lut(9, 6, 4, n, seed=n) for n in (2, 3)]
    O = [e(4, 6), e(4, 6)]
    yield "tc_lut", [[d(t) for t, _ in T], [d(i) for _, i in T], O], O


NAMES = {"tc_tbmm": "tbmm", "tc_tbmm_ws": "tbmm_ws", "tc_mlp_fcrelu": "mlp", "tc_group_conv": "gconv", "tc_kron": "kron", "tc_sconv2d": "sconv",
         "tc_lut": "lut"}


def test_what_is_not_on_a_gpu_is_left_to_the_general_path():
    tc.lib()
    for name, args, _ in _calls("cpu"):
        assert getattr(tc._FAST, NAMES[name])(0, *args, None) == -1  # (entry 0: a call would crash)
        with pytest.raises((TypeError, ValueError)):
            getattr(tc, name)(*args)
        for bad in (None, 3, "x", [], [None], object()):
            assert getattr(tc._FAST, NAMES[name])(0, *[bad] * len(args), None) == -1
        assert getattr(tc._FAST, NAMES[name])(0) == -1 and getattr(tc._FAST, NAMES[name])() == -1


@pytest.mark.gpu
def test_the_same_results_by_both_ways(monkeypatch):
    tc.lib()
    ways = []
    for fast in (tc._FAST, None):
        monkeypatch.setattr(tc, "_FAST", fast)
        got = []
        for name, args, outs in _calls("cuda"):
            getattr(tc, name)(*args)
            getattr(tc, name)(*args, stream=torch.cuda.current_stream().cuda_stream)
            got += [o.clone() for o in outs]
        ways.append(got)
    assert all(torch.equal(a, b) and not bool(a.isnan().any()) for a, b in zip(*ways))


@pytest.mark.gpu
def test_the_stream_of_a_call(monkeypatch):
    """Recorded on the stream that is current, in a graph that no other stream's work would enter."""
    tc.lib()
    for name, args, outs in _calls("cuda"):
        getattr(tc, name)(*args)
        torch.cuda.synchronize()
        want = [o.clone() for o in outs]
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            assert getattr(tc._FAST, NAMES[name])(tc._AT[name], *args, None) == 0
        for _ in range(2):
            for o in outs:
                o.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(o, w) for o, w in zip(outs, want)), name


@pytest.mark.gpu
def test_wrong_tensors_are_refused_as_before():
    tc.lib()
    X, Y, Z = torch.rand(2, 4, 8, device="cuda"), torch.rand(2, 6, 8, device="cuda"), torch.empty(2, 4, 6, device="cuda")
    with pytest.raises(TypeError):
        tc.tc_tbmm(X.double(), Y, Z)
    with pytest.raises(TypeError):
        tc.tc_tbmm(X.cpu(), Y, Z)
    with pytest.raises(ValueError):
        tc.tc_tbmm(X, Y, torch.empty(2, 6, 4, device="cuda"))
    with pytest.raises(ValueError):
        tc.tc_tbmm(X, Y, torch.empty(2, 6, 4, device="cuda").transpose(1, 2))
    with pytest.raises(tc.TcError):
        tc.tc_tbmm(X, Y, torch.empty(49, device="cuda")[1:].view(2, 4, 6))  # not 16-byte aligned
    with pytest.raises(tc.TcError):
        tc.tc_mlp_fcrelu(X[0], [Y[0], torch.rand(3, 6, device="cuda")], [torch.rand(6, device="cuda"), torch.rand(3, device="cuda")],
                         [None, torch.empty(4, 3, device="cuda")], None)  # no workspace
    with pytest.raises((TypeError, AttributeError)):
        tc.tc_kron(None, X[0], X, Z)
    tc.tc_tbmm(torch.nn.Parameter(X), Y, Z)
    assert torch.allclose(Z, X @ Y.transpose(1, 2), atol=1e-5)
    with pytest.raises(Exception):  # a wrapper has no memory of its own: refused, not read
        torch.func.vmap(lambda x: (tc.tc_tbmm(x, Y, Z), x)[1])(torch.rand(3, 2, 4, 8, device="cuda"))
