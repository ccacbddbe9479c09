"""The functions of the package go through native code for plain tensors on the current GPU (csrc/fle_torch.cpp) and through the
classes of the binding for everything else: the same results bit for bit, the same errors, and a defined answer (None: not for
here) for every kind of argument that the native code leaves alone."""
import threading

import pytest
import torch

from paper_2511_16964_amd import attention, binding, fused_linear_epilogue, grouped_fused_linear_epilogue, inputs, transformer_layer

from parity import dev_epilogue, to_dev

pytestmark = pytest.mark.gpu

F32, BF16, F16, F8 = torch.float32, torch.bfloat16, torch.float16, torch.float8_e4m3fn


@pytest.fixture(scope="module")
def native():
    return binding._load_native()


@pytest.mark.parametrize("dtype,M,N,K,kinds,kw", [
    (F32, 64, 256, 256, ["bias", "gelu_erf"], {}), (BF16, 33, 130, 72, ["bias", "relu", "scale", "residual"], {}), (F16, 1, 1, 1, ["bias"], {}),
    (BF16, 200, 520, 512, ["bias", "residual", "store", "layernorm"], {}), (F16, 70, 97, 83, ["bias", "softmax"], {}), (BF16, 19, 264, 128, ["scale", "logsumexp"], {}),
    (BF16, 2, 1024, 1024, ["bias", "gelu_tanh"], dict(ln_pre=True)), (F8, 130, 260, 256, ["scale", "bias", "residual"], {}), (F8, 77, 132, 256, ["bias", "layernorm"], dict(mx=True)),
    (F32, 5, 300, 129, [], {}),
])
def test_linear_is_the_same_as_through_the_class(native, dtype, M, N, K, kinds, kw):
    prob = inputs.random_problem(201, M, N, K, dtype, kinds, **kw)
    print("[case]", dtype, M, N, K, kinds, flush=True)
    x, w, b = to_dev(prob.x), to_dev(prob.w), to_dev(prob.b)
    ep = dev_epilogue(prob.epilogue)
    want = binding.Call(x, w, b, ep).run()
    stores = [e[1] for e in ep if e[0] == "store"]
    kept = [t.clone() for t in stores]
    for t in stores:
        t.fill_(float("nan"))
    got = native.linear(x, w, b, ep, None)
    assert got is not None and got.dtype == want.dtype and got.shape == want.shape and got.stride() == want.stride()
    assert torch.equal(got, want) and all(torch.equal(a, c) for a, c in zip(stores, kept))
    assert torch.equal(native.linear(x, w, b, tuple(ep), None), want)
    # into a buffer with longer rows
    if want.dim() == 2:
        buf = torch.full((M, N + 7), 3.0, dtype=want.dtype, device="cuda:0")
        out = buf[:, :N]
        assert native.linear(x, w, b, ep, out) is out and torch.equal(out, want) and (buf[:, N:] == 3.0).all()


def test_strided_operands_and_other_streams(native):
    prob = inputs.random_problem(203, 90, 260, 192, BF16, ["bias", "residual", "layernorm"])
    x, w, b, ep = to_dev(prob.x), to_dev(prob.w), to_dev(prob.b), dev_epilogue(prob.epilogue)
    want = binding.Call(x, w, b, ep).run()
    wide = lambda t: torch.nn.functional.pad(t, (0, 8))[:, :t.shape[1]]
    ep2 = [("residual", wide(e[1])) if e[0] == "residual" else e for e in ep]
    assert torch.equal(native.linear(wide(x), wide(w), b, ep2, None), want)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        got = [native.linear(x, w, b, ep, None) for _ in range(8)]   # (scratch of one call is the next one's: the same stream)
    side.synchronize()
    assert all(torch.equal(g, want) for g in got)
    results = []

    def worker():
        with torch.cuda.stream(torch.cuda.Stream()):
            r = [fused_linear_epilogue(x, w, b, ep) for _ in range(20)]
            torch.cuda.current_stream().synchronize()
            results.append(all(torch.equal(t, want) for t in r))
    torch.cuda.synchronize()
    threads = [threading.Thread(target=worker) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert results == [True] * 4


def test_grouped_attention_and_layer_are_the_same(native):
    torch.manual_seed(5)
    n = lambda *s: torch.randn(s, device="cuda:0").to(BF16)
    x, w, b = n(300, 128), n(5, 96, 128), n(5, 96)
    off = torch.tensor([0, 10, 10, 150, 299, 300], device="cuda:0")
    for bias in (b, b[0].contiguous(), None):
        ep = ([("bias",)] if bias is not None else []) + [("gelu_tanh",)]
        assert torch.equal(native.grouped_linear(x, w, bias, ep, None, off), binding.Call(x, w, bias, ep, offsets=off).run())
    qkv = n(2, 70, 3, 4, 64)
    q, k, v = qkv[:, :, 0], qkv[:, :, 1], qkv[:, :, 2]
    for causal in (False, True, 0, 1, 7):
        for scale in (None, 0.25):
            assert torch.equal(native.attention(q, k, v, causal, scale), binding.AttentionCall(q, k, v, causal, scale).run())
    k2, v2 = n(3, 1000, 4, 128), n(3, 1000, 4, 128)   # keys cut into ranges
    assert torch.equal(native.attention(n(3, 1, 4, 128).copy_(k2[:, :1]), k2, v2, 1, None), binding.AttentionCall(k2[:, :1].contiguous(), k2, v2, 1).run())
    C, F = 128, 512
    args = [n(2, 50, C), n(2, 50, C), n(3 * C, C) / 11, n(3 * C), n(C, C) / 11, None, 2, True, (n(C), None, 1e-5), n(F, C) / 11, n(F), n(C, F) / 22, n(C), (n(C), n(C), 1e-5)]
    got, want = native.transformer_layer(*args), binding.TransformerLayerCall(*args).run()
    assert len(got) == 2 and all(torch.equal(a, c) for a, c in zip(got, want))


class Tagged(torch.Tensor):
    pass


def test_what_the_native_code_leaves_alone(native):
    x, w, b = (torch.randn(s, device="cuda:0").to(BF16) for s in ((8, 64), (32, 64), (32,)))
    ep = [("bias",)]
    want = binding.Call(x, w, b, ep).run()
    none = [
        (x.cpu(), w, b, ep, None), (x.as_subclass(Tagged), w, b, ep, None), (x.float(), w, b, ep, None), (x, w, b.float(), ep, None), (x, w, b[:31], ep, None),
        (x, w.t().contiguous().t(), b, ep, None), (x[:, ::2], w[:, ::2], b, ep, None), (x[:0], w, b, ep, None), (x[0], w, b, ep, None), (x, w, b, [("gone",)], None),
        (x, w, b, ep, torch.empty(8, 31, device="cuda:0", dtype=BF16)), (x, w, b, ep, torch.empty(8, 32, device="cuda:0")), (x, w, b, [["bias"]], None), (x, w, b, [("scale",)], None),
        (x, w, b, [("scale", torch.tensor(2.0))], None), (x, w, b, [("layernorm", None, None)], None), (x, w, b, [("residual", x)], None), (x, w, b, [("scale", float("nan"))], None),
        (x, w, b, [("bias",)] * 9, None), (x, w, b, [("softmax",)] * 3, None), (x, w, b, iter(ep), None), (None, w, b, ep, None), (x, w, None, ep, None),
    ]
    for args in none:
        assert native.linear(*args) is None
    # they go on to the class: its errors, or its results
    for args, err in ((none[0], RuntimeError), (none[2], TypeError), (none[3], TypeError), (none[4], ValueError), (none[5], ValueError), (none[9], KeyError),
                      (none[10], ValueError), (none[11], TypeError), (none[16], ValueError), (none[17], binding.FleError), (none[18], ValueError), (none[19], binding.FleError), (none[22], binding.FleError)):
        with pytest.raises(err):
            fused_linear_epilogue(*args[:4], out=args[4])
    assert torch.equal(fused_linear_epilogue(x.as_subclass(Tagged), w, b, ep).as_subclass(torch.Tensor), want)
    assert fused_linear_epilogue(x[:0], w, b, ep).shape == (0, 32)
    assert torch.equal(fused_linear_epilogue(x, w, b, ep, variant="general"), binding.Call(x, w, b, ep, variant="general").run())
    class Mode(torch.utils._python_dispatch.TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))
    with Mode():
        assert native.linear(x, w, b, ep, None) is None
        assert torch.equal(fused_linear_epilogue(x, w, b, ep), want)
    assert torch.func.vmap(lambda t: torch.tensor(native.linear(t, w, b, ep, None) is None), randomness="different")(x[None]).all()
    with pytest.raises(Exception):
        grouped_fused_linear_epilogue(x, w[None], b, torch.tensor([0, 8]), ep)   # offsets on the host
    q = torch.randn(1, 4, 2, 64, device="cuda:0")
    assert native.attention(q, q, q, 1, None) is None and native.attention(q.half(), q.half(), q.half(), -1, None) is None
    with pytest.raises(binding.FleError):
        attention(q, q, q, 1)
    assert native.transformer_layer(*[None] * 14) is None
    with pytest.raises(Exception):
        transformer_layer(*[None] * 14)


def test_captured_calls_replay(native):
    prob = inputs.random_problem(207, 640, 1000, 2048, BF16, ["bias", "gelu_tanh", "layernorm"])   # K split, row pass: scratch memory
    x, w, b, ep = to_dev(prob.x), to_dev(prob.w), to_dev(prob.b), dev_epilogue(prob.epilogue)
    out = torch.empty(640, 1000, device="cuda:0", dtype=BF16)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        fused_linear_epilogue(x, w, b, ep, out=out)
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        fused_linear_epilogue(x, w, b, ep, out=out)
        fused_linear_epilogue(x, w, b, ep, out=out)
    for i in range(3):
        x.copy_(torch.randn(640, 2048, device="cuda:0"))
        want = binding.Call(x, w, b, ep).run()
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), i


def test_operands_outlive_a_list_that_changes_during_the_call(native):
    """A list is emptied while it is read (here by a factor's own conversion; another thread can do it as well): the call goes
    by the entries that it began with, and memory of their tensors is nobody else's until it is enqueued."""
    prob = inputs.random_problem(211, 96, 260, 128, BF16, ["bias", "residual", "layernorm"])
    x, w, b, ep = to_dev(prob.x), to_dev(prob.w), to_dev(prob.b), dev_epilogue(prob.epilogue)
    want = binding.Call(x, w, b, [("scale", 2.0)] + ep).run()
    held, others = [], []

    class Factor(int):
        def __float__(self):
            shapes = [t.shape for e in held for t in e if isinstance(t, torch.Tensor)]
            held.clear()
            others.extend(torch.full(s, 1000.0, dtype=BF16, device="cuda:0") for s in shapes for _ in range(2))
            return 2.0

    for tensors_first in (False, True):
        own = [tuple(t.clone() if isinstance(t, torch.Tensor) else t for t in e) for e in ep]
        tail = [("scale", Factor(2))] if tensors_first else []
        held[:] = ([] if tensors_first else [("scale", Factor(2))]) + own[:2] + tail + own[2:]
        expect = binding.Call(x, w, b, ep[:2] + [("scale", 2.0)] + ep[2:]).run() if tensors_first else want
        del own
        got = native.linear(x, w, b, held, None)
        assert held == [] and torch.equal(got, expect)
