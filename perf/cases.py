"""Workloads of the library's six operators, as a program that uses them calls them.

Sizes and distributions are those of ``paper_1802_04730_amd/inputs.py``, of the benchmark and of the tests where
these have one, and generic ones elsewhere: real models rarely come in multiples of 16.  Inputs are drawn on the GPU,
outputs and workspaces belong to the caller and are kept, as the C ABI means them to be.
"""
from __future__ import annotations

import torch

from paper_1802_04730_amd import inputs, tc355


def listed():
    return [
        # Factorization-machine interactions: many tiny products, the benchmark's tbmm; latency and launch count
        dict(name="tbmm_500", op="tbmm", B=500, N=26, M=72, K=26),
        # the same at serving scale with feature counts that divide nothing: streaming, unaligned rows
        dict(name="tbmm_odd", op="tbmm", B=4000, N=27, M=61, K=35),
        # one wide layer against a large weight matrix, workspace kept between calls (the paper's largest tmm)
        dict(name="tmm_large", op="tbmm", B=1, N=128, M=16384, K=4096),
        # the production chain of three fully connected layers, batch 128 (the benchmark's MLP)
        dict(name="mlp_128", op="mlp", batch=128, dims="1024,1024,512,256", keep=True),
        # scoring with widths as feature engineering leaves them; only the last output is wanted
        dict(name="mlp_ragged", op="mlp", batch=300, dims="429,1000,600,250", keep=False),
        # the benchmark's grouped convolution: a full ResNeXt-style layer at batch 32, image with its border
        dict(name="gconv_58", op="gconv", N=32, G=32, C=16, F=16, H=58, W=58, KH=3, KW=3, bias=True),
        # a layer of the paper's table further down the network: smaller image, narrower groups
        dict(name="gconv_28", op="gconv", N=32, G=32, C=8, F=8, H=28, W=28, KH=3, KW=3, bias=True),
        # a layer of no particular size: channels, filters and image sides that fit no tile
        dict(name="gconv_odd", op="gconv", N=16, G=24, C=12, F=20, H=33, W=45, KH=3, KW=3, bias=False),
        # Kronecker-factored layer, the benchmark's
        dict(name="kron_256", op="kron", B=256, I=64, K=64, J=64, L=64),
        # the same with factors chosen from a layer whose widths factor unevenly
        dict(name="kron_odd", op="kron", B=200, I=48, K=50, J=75, L=36),
        # down-sampling layer of a convolution network, batch 32 (the benchmark's strided convolution)
        dict(name="sconv_56", op="sconv", N=32, C=64, F=128, H=56, W=56, KH=3, KW=3, sh=2, sw=2, bias=True),
        # two embedding tables of the paper's production model, fresh rows all over a table far beyond any cache
        dict(name="lut_2", op="lut", tables=2, E=10_000_000, D=64, B=128, L=50),
    ]


def _log(rng, lo, hi):
    """An integer whose logarithm is uniform over [lo, hi]."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def _draw_tbmm(rng):
    return dict(op="tbmm", B=_log(rng, 8, 32000), N=rng.randint(8, 100), M=rng.randint(8, 100), K=rng.randint(8, 100))


def _draw_tmm(rng):
    # weight matrices of fully connected layers without bias; blocks of 128 rows are the commonest batch
    n = rng.choice([128, 128, 256, _log(rng, 16, 512)])
    step = rng.choice([1, 4, 64])
    m, k = (max(step, _log(rng, 64, 16384) // step * step), max(step, _log(rng, 64, 4096) // step * step))
    return dict(op="tbmm", B=1, N=n, M=m, K=k)


def _draw_mlp(rng):
    layers = rng.randint(1, 4)
    if rng.random() < 0.5:
        dims = [rng.choice([128, 256, 512, 1024]) for _ in range(layers + 1)]
    else:
        dims = [_log(rng, 16, 2048) for _ in range(layers + 1)]
    return dict(op="mlp", batch=_log(rng, 1, 2048), dims=",".join(map(str, dims)), keep=rng.random() < 0.5)


def _draw_gconv(rng):
    n, g, bias = _log(rng, 1, 32), _log(rng, 1, 32), rng.random() < 0.5
    if rng.random() < 0.5:  # layers of ResNeXt-like networks
        c = rng.choice([4, 8, 16, 32])
        h = rng.choice([56, 28, 14, 7]) + rng.choice([0, 0, 2])
        return dict(op="gconv", N=n, G=rng.choice([g, 32]), C=c, F=c, H=h, W=h, KH=3, KW=3, bias=bias)
    k = rng.choice([1, 3, 3, 3, 5])
    return dict(op="gconv", N=n, G=g, C=rng.randint(2, 40), F=rng.randint(2, 40), H=rng.randint(7, 64), W=rng.randint(7, 64),
                KH=k, KW=k, bias=bias)


def _draw_kron(rng):
    return dict(op="kron", B=_log(rng, 8, 2048), I=rng.randint(8, 100), K=rng.randint(8, 100), J=rng.randint(8, 100),
                L=rng.randint(8, 100))


def _draw_sconv(rng):
    k, s = rng.choice([1, 3, 3, 5, 7]), rng.choice([1, 2, 2])
    c, f = rng.choice([3, 64, 128, 256, _log(rng, 3, 256)]), rng.choice([64, 128, 256, _log(rng, 16, 256)])
    h = rng.choice([224, 56, 28, 14, rng.randint(7, 112)])
    return dict(op="sconv", N=_log(rng, 1, 32), C=c, F=f, H=h, W=rng.choice([h, rng.randint(7, 112)]), KH=k, KW=k, sh=s, sw=s,
                bias=rng.random() < 0.5)


def _draw_lut(rng):
    return dict(op="lut", tables=rng.randint(1, 4), E=_log(rng, 10_000, 10_000_000),
                D=rng.choice([16, 32, 64, 128, rng.randint(8, 200)]), B=_log(rng, 16, 4096), L=_log(rng, 1, 100))


# Most work a drawn case may have, per operator: no more than its listed cases take (flops, bytes).
_MOST = {"tbmm": (9e9, 2.2e8), "mlp": (4e9, 1e8), "gconv": (2.2e9, 3e8), "kron": (2e9, 1.5e8), "sconv": (4e9, 3e8),
         "lut": (1e9, 1.2e8)}


def draw(rng):
    kind = rng.choice([_draw_tbmm, _draw_tmm, _draw_mlp, _draw_gconv, _draw_kron, _draw_sconv, _draw_lut])
    while True:
        case = kind(rng)
        w = work(case)
        flops, nbytes = _MOST[case["op"]]
        if w["flops"] <= flops and w["bytes"] <= nbytes and w["flops"] >= 1e4:
            return case


def _dims(case):
    return [int(d) for d in case["dims"].split(",")]


class _Draws:
    """Tensors drawn on the GPU from one seeded generator."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))

    def normal(self, std, *shape):
        return torch.randn(shape, device="cuda", generator=self.g).mul_(std)

    def uniform(self, *shape):
        return torch.rand(shape, device="cuda", generator=self.g).mul_(2.0).sub_(1.0)

    def index(self, hi, *shape):
        return torch.randint(0, hi, shape, device="cuda", generator=self.g, dtype=torch.int32)


def _empty(*shape):
    return torch.empty(shape, device="cuda")


def prepare(case, seed):
    d, op = _Draws(seed), case["op"]
    if op == "tbmm":
        B, N, M, K = (case[k] for k in "BNMK")
        nbytes = tc355.tc_tbmm_workspace_bytes(B, N, M, K)
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None
        return dict(op=op, X=d.uniform(B, N, K), Y=d.uniform(B, M, K), Z=_empty(B, N, M), ws=ws)
    if op == "mlp":
        dims, batch = _dims(case), case["batch"]
        n = len(dims) - 1
        nbytes = tc355.tc_mlp_fcrelu_workspace_bytes(batch, dims)
        return dict(op=op, I=d.normal(1.0, batch, dims[0]),
                    # weights of a layer scale with its fan-in, so that activations keep their size down the chain
                    W=[d.normal((2.0 / dims[l]) ** 0.5, dims[l + 1], dims[l]) for l in range(n)],
                    b=[d.normal(0.01, dims[l + 1]) for l in range(n)],
                    O=[_empty(batch, dims[l + 1]) if case["keep"] or l == n - 1 else None for l in range(n)],
                    ws=torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None)
    if op == "gconv":
        N, G, C, F, H, W, KH, KW = (case[k] for k in ("N", "G", "C", "F", "H", "W", "KH", "KW"))
        return dict(op=op, I=d.normal(1.0, N, G, C, H, W), Wt=d.normal(0.05, G, F, C, KH, KW),
                    b=d.normal(0.05, G * F) if case["bias"] else None, O=_empty(N, G, F, H - KH + 1, W - KW + 1))
    if op == "kron":
        B, I, K, J, L = (case[k] for k in "BIKJL")
        return dict(op=op, W1=d.normal(0.125, I, K), W2=d.normal(0.125, J, L), X=d.normal(0.125, B, K, L), Y=_empty(B, I, J))
    if op == "sconv":
        N, C, F, H, W, KH, KW, sh, sw = (case[k] for k in ("N", "C", "F", "H", "W", "KH", "KW", "sh", "sw"))
        return dict(op=op, I=d.normal(1.0, N, C, H, W), Wt=d.normal(0.05, F, C, KH, KW), b=d.normal(0.05, F) if case["bias"] else None,
                    O=_empty(N, F, (H - KH) // sh + 1, (W - KW) // sw + 1), sh=sh, sw=sw)
    T, E, D, B, L = (case[k] for k in ("tables", "E", "D", "B", "L"))
    return dict(op=op, T=[d.normal(1.0, E, D) for _ in range(T)], Idx=[d.index(E, B, L) for _ in range(T)],
                O=[_empty(B, D) for _ in range(T)])


def run(state):
    op = state["op"]
    if op == "tbmm":
        if state["ws"] is None:
            tc355.tc_tbmm(state["X"], state["Y"], state["Z"])
        else:
            tc355.tc_tbmm_ws(state["X"], state["Y"], state["Z"], state["ws"])
        return state["Z"]
    if op == "mlp":
        tc355.tc_mlp_fcrelu(state["I"], state["W"], state["b"], state["O"], state["ws"])
        return [o for o in state["O"] if o is not None]
    if op == "gconv":
        tc355.tc_group_conv(state["I"], state["Wt"], state["b"], state["O"])
        return state["O"]
    if op == "kron":
        tc355.tc_kron(state["W1"], state["W2"], state["X"], state["Y"])
        return state["Y"]
    if op == "sconv":
        tc355.tc_sconv2d(state["I"], state["Wt"], state["b"], state["O"], state["sh"], state["sw"])
        return state["O"]
    tc355.tc_lut(state["T"], state["Idx"], state["O"])
    return state["O"]


def work(case):
    op = case["op"]
    size = {k: v for k, v in case.items() if k not in ("name", "op", "bias", "keep", "tables")}
    if op == "tbmm":
        return dict(flops=inputs.flops_tbmm(**size), bytes=inputs.bytes_tbmm(**size))
    if op == "mlp":
        dims, batch = _dims(case), case["batch"]
        inner = 0 if case["keep"] else 4 * batch * sum(dims[1:-1])  # outputs that are not asked for are not written
        return dict(flops=inputs.flops_mlp(batch, dims), bytes=inputs.bytes_mlp(batch, dims) - inner)
    if op == "gconv":
        return dict(flops=inputs.flops_gconv(**size), bytes=inputs.bytes_gconv(**size))
    if op == "kron":
        B, I, K, J, L = (case[k] for k in "BIKJL")
        # either factor may be applied first; the cheaper order counts
        return dict(flops=min(2 * B * I * L * (K + J), 2 * B * K * J * (L + I)), bytes=inputs.bytes_kron(**size))
    if op == "sconv":
        return dict(flops=inputs.flops_sconv2d(**size), bytes=inputs.bytes_sconv2d(**size))
    T = case["tables"]
    return dict(flops=T * inputs.flops_lut(**size), bytes=T * inputs.bytes_lut(**size))


def tolerance(case):
    # Every operator sums exactly or in 64 bits and rounds each output once to fp32: against the same path in float64
    # all of the cases above and thirty drawn ones measure 2.4e-8 .. 2.6e-8 (2-norm) and at most 6.3e-8 (largest, that
    # is one rounding).  Four times that.
    return {"rel": 1e-7, "max": 2.5e-7}
