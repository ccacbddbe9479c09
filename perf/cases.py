"""The calls whose speed is followed from one version of the library to the next.

Every case is a piece of work that a program hands to the package's public entry points, as README.md shows them:
the smallest call, where the host and the launch count; one token or a handful of rows against whole weight
matrices; ordinary and large layers in each operand dtype; ragged sizes; expert-routed rows; attention over a
sequence and attention of one new token over kept keys; whole perceptrons, blocks and transformer layers.
"""
from __future__ import annotations

import math

import torch

from paper_2511_16964_amd import attention, fused_linear_epilogue, grouped_fused_linear_epilogue, mlp_chain, transformer_layer

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16, "f8": torch.float8_e4m3fn, "mx": torch.float8_e4m3fn}
EPS = 1e-5


def listed():
    return [
        # one small fp32 layer (a head of a small model): launch and host latency
        dict(name="tiny_f32", kind="linear", dtype="f32", chain="bias_gelu_erf", M=64, N=256, K=256),
        # one token through a block's normalisation and projection: decoding at batch 1
        dict(name="token_norm_bf16", kind="linear", dtype="bf16", chain="norm_bias_gelu_erf", M=1, N=4096, K=4096),
        # a perceptron at batch 1, eight layers in one launch: every weight is read once
        dict(name="perceptron_f32", kind="chain", dtype="f32", weights="f32", width=4096, layers=8),
        # a decoding batch against a vocabulary-sized matrix, row softmax: bound by the weights
        dict(name="vocabulary_bf16", kind="linear", dtype="bf16", chain="softmax", M=32, N=32768, K=8192),
        # an ordinary square layer with an elementwise tail
        dict(name="layer_bf16", kind="linear", dtype="bf16", chain="bias_relu_scale_residual", M=4096, N=4096, K=4096),
        # the same layer with x and W stored in fp8
        dict(name="layer_f8", kind="linear", dtype="f8", chain="scale_bias_relu_scale_residual", M=4096, N=4096, K=4096),
        # sizes that are multiples of nothing: rows, columns and the reduction all odd
        dict(name="ragged_f16", kind="linear", dtype="f16", chain="bias_residual_layernorm", M=1999, N=4099, K=3071),
        # a transformer's perceptron block over a large batch of tokens
        dict(name="mlp_block_bf16", kind="mlp", dtype="bf16", M=16384, width=4096, hidden=16384),
        # rows routed to experts, a prefill batch: one grouped call
        dict(name="experts_bf16", kind="grouped", dtype="bf16", M=32768, G=32, N=4096, K=4096),
        # one new token per sequence against the keys and values kept from earlier ones
        dict(name="attention_decode_bf16", kind="attention", dtype="bf16", B=4, T=1, Tk=8192, H=16, D=128, causal=1),
        # many short unmasked sequences of an odd length (image patches)
        dict(name="attention_patches_bf16", kind="attention", dtype="bf16", B=32, T=197, Tk=197, H=12, D=64, causal=0),
        # a whole pre-norm transformer layer over 16 sequences of 2048 tokens
        dict(name="transformer_bf16", kind="layer", dtype="bf16", B=16, T=2048, C=2048, H=16, F=8192),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _up(v, m):
    return max(m, (v + m - 1) // m * m)


def draw(rng):
    kind = rng.choice(["linear"] * 6 + ["mlp", "grouped", "chain", "attention", "attention", "layer"])
    if kind == "linear":
        dtype = rng.choice(["bf16", "bf16", "bf16", "f16", "f32", "f8", "mx"])
        M, N, K = _log(rng, 1, 16384), _log(rng, 128, 32768), _log(rng, 128, 16384)
        form = rng.choice(["whole", "whole", "odd_n", "odd"])
        if dtype in ("f8", "mx"):
            K, N = _up(K, 16 if dtype == "f8" and form != "whole" else 128), (N | 1 if form == "odd_n" else _up(N, 16))
            chain = rng.choice(["scale_bias_relu_scale_residual", "bias_gelu_erf", "bias_residual_layernorm"])
        else:
            if form == "odd":
                N, K = N | 1, K | 1
            else:
                N, K = (N | 1 if form == "odd_n" else _up(N, 64)), _up(K, 64)
            chain = rng.choice(["bias_gelu_erf", "bias_relu_scale_residual", "bias_residual_layernorm", "bias_gelu_tanh_layernorm", "norm_bias_gelu_erf", "softmax", "bias_logsumexp"])
        cap = 2.7e11 if dtype == "f32" or K % 8 else 2.2e12
        M = max(1, min(M, int(cap / (2.0 * N * K))))
        return dict(kind=kind, dtype=dtype, chain=chain, M=M, N=N, K=K)
    if kind == "mlp":
        width = 128 * rng.randint(4, 32)
        return dict(kind=kind, dtype=rng.choice(["bf16", "f16"]), M=_log(rng, 8, 16384), width=width, hidden=4 * width)
    if kind == "grouped":
        N, K, G = 64 * rng.randint(8, 64), 64 * rng.randint(8, 64), rng.choice([4, 8, 16, 32, 33])
        return dict(kind=kind, dtype=rng.choice(["bf16", "f16"]), M=_log(rng, 64, 32768), G=G, N=N, K=K)
    if kind == "chain":
        dtype = rng.choice(["f32", "bf16"])
        return dict(kind=kind, dtype=dtype, weights=rng.choice([dtype, "bf16"]), width=64 * rng.randint(4, 96), layers=rng.randint(2, 8))
    if kind == "attention":
        H, D = rng.choice([8, 12, 16, 25]), rng.choice([32, 64, 128, 128, 256])
        dtype = rng.choice(["bf16", "f16"])
        if rng.random() < 0.5:  # new tokens against kept keys
            T, Tk = rng.choice([1, 1, 1, 2, 5]), _log(rng, 64, 16384)
            B = max(1, min(_log(rng, 1, 64), (1 << 28) // (Tk * H * D)))
            return dict(kind=kind, dtype=dtype, B=B, T=T, Tk=Tk, H=H, D=D, causal=1)
        T = _log(rng, 32, 8192)
        B = max(1, min(_log(rng, 1, 64), int(1e12 / (4.0 * H * D * T * T))))
        return dict(kind=kind, dtype=dtype, B=B, T=T, Tk=T, H=H, D=D, causal=rng.choice([0, 1]))
    H, D = rng.choice([8, 12, 16]), rng.choice([64, 128])
    T = _log(rng, 64, 4096)
    return dict(kind="layer", dtype=rng.choice(["bf16", "f16"]), B=max(1, min(_log(rng, 1, 32), 32768 // T)), T=T, C=H * D, H=H, F=4 * H * D)


class _Inputs:
    """Random tensors of one seed, drawn on the GPU."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)

    def normal(self, shape, dtype, mean=0.0, std=1.0):
        return torch.empty(shape, device="cuda", dtype=torch.float32).normal_(mean, std, generator=self.gen).to(dtype)

    def uniform(self, shape, dtype, a):
        return torch.empty(shape, device="cuda", dtype=torch.float32).uniform_(-a, a, generator=self.gen).to(dtype)

    def affine(self, n, dtype):
        """gamma and beta of a LayerNorm."""
        return self.normal((n,), dtype, 1.0, 0.02), self.normal((n,), dtype, 0.0, 0.02)


def _to_f8(t):
    """A tensor in e4m3 with one scale for all of it."""
    scale = float(t.abs().max()) / 448.0
    return (t / scale).to(torch.float8_e4m3fn), scale


def _to_mx(t):
    """A matrix in e4m3 with one power-of-two scale (E8M0) per 32 consecutive elements of a row."""
    blocks = t.view(t.shape[0], -1, 32)
    _, e = torch.frexp(blocks.abs().amax(dim=2))
    e = (e - 1 - 8).clamp(-127, 127)
    q = torch.ldexp(blocks, -e.unsqueeze(2)).clamp(-448.0, 448.0)
    return q.reshape(t.shape).to(torch.float8_e4m3fn), (e + 127).to(torch.uint8).contiguous()


def _linear(case, inp):
    M, N, K, dt = case["M"], case["N"], case["K"], DTYPES[case["dtype"]]
    f8 = dt == torch.float8_e4m3fn
    io, a = (torch.bfloat16 if f8 else dt), 1.0 / math.sqrt(K)
    ops = case["chain"]
    x, w = inp.normal((M, K), torch.float32 if f8 else dt, 0.25 if "norm_bias" in ops else 0.0), inp.uniform((N, K), torch.float32 if f8 else dt, a)
    epilogue, factor = [], 0.5
    if ops.startswith("norm_"):
        epilogue.append(("layernorm_pre",) + inp.affine(K, io) + (EPS,))
        ops = ops[5:]
    if case["dtype"] == "mx":
        (x, sx), (w, sw) = _to_mx(x), _to_mx(w)
        epilogue.append(("mxscale", sx, sw))
    elif case["dtype"] == "f8":
        (x, sx), (w, sw) = _to_f8(x), _to_f8(w)
        epilogue.append(("scale", sx * sw))
    ops = ops.replace("gelu_", "gelu-").split("_")
    if ops[0] == "scale":  # (the operands' own scale, in the list already)
        ops = ops[1:]
    for op in ops:
        if op in ("gelu-erf", "gelu-tanh"):
            epilogue.append((op.replace("-", "_"),))
        elif op == "scale":
            epilogue.append(("scale", factor))
        elif op == "residual":
            epilogue.append(("residual", inp.normal((M, N), io)))
        elif op == "layernorm":
            epilogue.append(("layernorm",) + inp.affine(N, io) + (EPS,))
        else:
            epilogue.append((op,))
    return dict(x=x, w=w, b=inp.uniform((N,), io, a) if ("bias",) in epilogue else None, epilogue=epilogue)


def prepare(case, seed):
    inp, kind, dt = _Inputs(seed), case["kind"], DTYPES[case["dtype"]]
    state = dict(kind=kind, case=dict(case))
    if kind == "linear":
        state.update(_linear(case, inp))
    elif kind == "mlp":
        M, C, F = case["M"], case["width"], case["hidden"]
        state.update(x=inp.normal((M, C), dt), w1=inp.uniform((F, C), dt, C ** -0.5), b1=inp.uniform((F,), dt, C ** -0.5),
                     w2=inp.uniform((C, F), dt, F ** -0.5), b2=inp.uniform((C,), dt, F ** -0.5), ln=inp.affine(C, dt) + (EPS,))
    elif kind == "grouped":
        M, G, N, K = case["M"], case["G"], case["N"], case["K"]
        # an imbalanced router: rows spread over the groups by random probabilities (Dirichlet(1))
        host = torch.Generator().manual_seed(seed)
        p = torch.empty(G).exponential_(generator=host)
        counts = torch.bincount(torch.multinomial(p, M, replacement=True, generator=host), minlength=G)
        offsets = torch.zeros(G + 1, dtype=torch.int64)
        offsets[1:] = counts.cumsum(0)
        state.update(x=inp.normal((M, K), dt), w=inp.uniform((G, N, K), dt, K ** -0.5), b=inp.uniform((G, N), dt, K ** -0.5), offsets=offsets.cuda())
    elif kind == "chain":
        k, wdt = case["width"], DTYPES[case["weights"]]
        a = math.sqrt(6.0 / k)
        state.update(x=inp.normal((1, k), dt), ws=[inp.uniform((k, k), wdt, a) for _ in range(case["layers"])],
                     bs=[inp.uniform((k,), dt, 0.1) for _ in range(case["layers"])])
    elif kind == "attention":
        B, T, Tk, H, D = (case[n] for n in ("B", "T", "Tk", "H", "D"))
        if T == Tk:  # the three thirds of one projection's output
            qkv = inp.normal((B, T, 3, H, D), dt)
            state.update(q=qkv[:, :, 0], k=qkv[:, :, 1], v=qkv[:, :, 2])
        else:
            state.update(q=inp.normal((B, T, H, D), dt), k=inp.normal((B, Tk, H, D), dt), v=inp.normal((B, Tk, H, D), dt))
    else:
        B, T, C, F = (case[n] for n in ("B", "T", "C", "F"))
        s = C ** -0.5
        state.update(x=inp.normal((B, T, C), dt), n=inp.normal((B, T, C), dt), w_qkv=inp.normal((3 * C, C), dt, 0.0, s), b_qkv=inp.uniform((3 * C,), dt, 0.1),
                     w_o=inp.normal((C, C), dt, 0.0, s), b_o=inp.uniform((C,), dt, 0.1), w1=inp.uniform((F, C), dt, s), b1=inp.uniform((F,), dt, s),
                     w2=inp.uniform((C, F), dt, F ** -0.5), b2=inp.uniform((C,), dt, F ** -0.5), mid=inp.affine(C, dt) + (EPS,), out=inp.affine(C, dt) + (EPS,))
    return state


def run(state):
    s, kind = state, state["kind"]
    if kind == "linear":
        return fused_linear_epilogue(s["x"], s["w"], s["b"], s["epilogue"])
    if kind == "mlp":
        h = fused_linear_epilogue(s["x"], s["w1"], s["b1"], [("bias",), ("gelu_erf",)])
        return fused_linear_epilogue(h, s["w2"], s["b2"], [("bias",), ("residual", s["x"]), ("layernorm",) + s["ln"]])
    if kind == "grouped":
        return grouped_fused_linear_epilogue(s["x"], s["w"], s["b"], s["offsets"], [("bias",), ("gelu_tanh",)])
    if kind == "chain":
        return mlp_chain(s["x"], s["ws"], s["bs"], ["relu"] * len(s["ws"]))
    if kind == "attention":
        return attention(s["q"], s["k"], s["v"], causal=s["case"]["causal"])
    return transformer_layer(s["x"], s["n"], s["w_qkv"], s["b_qkv"], s["w_o"], s["b_o"], s["case"]["H"], True, s["mid"], s["w1"], s["b1"], s["w2"], s["b2"], s["out"])


def work(case):
    kind = case["kind"]
    es = {"f32": 4, "f8": 1, "mx": 1}.get(case["dtype"], 2)
    if kind == "linear":
        M, N, K, ops = case["M"], case["N"], case["K"], case["chain"]
        io = 2 if es == 1 else es
        n = (M * K + N * K) * es + (M if ops.endswith("logsumexp") else M * N) * io + ("bias" in ops) * N * io + ("residual" in ops) * M * N * io
        n += ops.endswith("layernorm") * 2 * N * io + ops.startswith("norm_") * 2 * K * io + (case["dtype"] == "mx") * (M + N) * K // 32
        return dict(bytes=n, flops=2 * M * N * K)
    if kind == "mlp":
        M, C, F = case["M"], case["width"], case["hidden"]
        return dict(bytes=(2 * M * C + 2 * C * F + F + 3 * C) * es, flops=4 * M * C * F)
    if kind == "grouped":
        M, G, N, K = case["M"], case["G"], case["N"], case["K"]
        return dict(bytes=(M * K + M * N + min(G, M) * (N * K + N)) * es + 8 * (G + 1), flops=2 * M * N * K)
    if kind == "chain":
        k, n, ws = case["width"], case["layers"], {"f32": 4}.get(case["weights"], 2)
        return dict(bytes=n * k * k * ws + (n + 2) * k * es, flops=2 * n * k * k)
    if kind == "attention":
        B, T, Tk, H, D = (case[n] for n in ("B", "T", "Tk", "H", "D"))
        pairs = T * Tk - (T * (T - 1) // 2 if case["causal"] else 0)
        return dict(bytes=2 * B * H * D * (T + Tk) * es, flops=4 * B * H * D * pairs)
    M, C, F, T = case["B"] * case["T"], case["C"], case["F"], case["T"]
    return dict(bytes=(4 * M * C + 4 * C * C + 2 * C * F + F + 9 * C) * es, flops=2 * M * C * (4 * C + 2 * F) + 4 * case["B"] * C * (T * (T + 1) // 2))


def tolerance(case):
    """Four times the largest error seen against the same composition in float64 (relative 2-norm): 3.8e-7 on fp32
    operands, 3.7e-4 on fp16, 2.9e-3 on bf16 (outputs rounded once to 2^-9, row statistics and stored intermediates
    included), 4.5e-3 on bf16 perceptrons, whose activations are rounded after every layer."""
    if case["dtype"] == "f32":
        return {"rel": 1.6e-6}
    if case["dtype"] == "f16":
        return {"rel": 1.5e-3}
    return {"rel": 1.8e-2 if case["kind"] == "chain" else 1.2e-2}
