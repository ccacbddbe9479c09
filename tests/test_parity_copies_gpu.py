"""GPU parity of operands whose rows are no whole, aligned 16-byte chunks and that are copied into the workspace first
(fle_gemm tiled / thin / skinny kernels behind the copies), and of the same calls where the workspace is too small."""
import pytest
import torch

from paper_2511_16964_amd import binding, inputs

from parity import assert_close, dev_epilogue, oracle_rows, sample_rows, to_dev

pytestmark = pytest.mark.gpu

F32, BF16, F16 = torch.float32, torch.bfloat16, torch.float16


def place(t, pad, shift):
    """The matrix inside a larger NaN-filled buffer: a row stride of its columns + pad, a start shifted by `shift` elements."""
    rows, cols = t.shape
    buf = torch.full((rows * (cols + pad) + shift + 16,), float("nan"), dtype=t.dtype, device="cuda:0")
    view = buf[shift:shift + rows * (cols + pad)].view(rows, cols + pad)[:, :cols]
    view.copy_(t.to("cuda:0"))
    return view


def call_of(prob, x=(0, 0), w=(0, 0), **kw):
    out = torch.full((prob.M,) if prob.epilogue[-1][0] == "logsumexp" else (prob.M, prob.N), float("nan"), dtype=prob.x.dtype, device="cuda:0")
    return binding.Call(place(prob.x, *x), place(prob.w, *w), to_dev(prob.b), dev_epilogue(prob.epilogue), out=out, **kw)


def check(prob, call, copies):
    print("[case]", prob.M, prob.N, prob.K, prob.x.dtype, copies, flush=True)
    got = call.run()
    torch.cuda.synchronize()
    text = call.plan()
    assert text.endswith(" copies=" + copies) if copies else "copies" not in text, text
    rows = sample_rows(prob.M, 24)
    assert torch.isfinite(got.float()).all(), text
    assert_close(got.cpu()[rows], oracle_rows(prob, rows), prob.x.dtype, what=text)


@pytest.mark.parametrize("dtype", [F32, BF16, F16])
@pytest.mark.parametrize("M,N,K,kinds,f32,two_byte", [  # the kernel behind the copies (None: read as they are) for fp32 and for 2-byte operands
    (2047, 1030, 1001, ["bias", "relu"], "tiled", "tiled"),            # K one element into a chunk
    (700, 3075, 1535, ["bias", "residual", "layernorm"], "tiled", "tiled"),  # and one short of it; row op, element-wise epilogue
    (650, 2051, 1537, ["bias", "softmax"], "tiled", "tiled"),
    (513, 1024, 2052, ["bias", "gelu_erf"], None, "tiled"),            # fp32: whole chunks; 2-byte: half a chunk over
    (300, 1500, 1001, ["bias", "logsumexp"], None, "tiled"),           # K split
    (1, 1023, 8191, ["bias"], "thin_dot", "thin_dot"),
    (4, 1030, 4095, ["bias", "softmax"], "thin_dot", "thin_dot"),
    (16, 1023, 16383, ["bias", "gelu_tanh"], None, "tiled"),           # K split in 16
    (16, 1023, 4095, ["bias", "gelu_tanh"], None, "thin_mfma"),
    (32, 1000, 4001, ["bias", "residual", "layernorm"], None, "thin_mfma"),  # (K = 2001 is faster read as it is)
    (5, 1025, 4001, ["bias", "logsumexp"], "thin_dot", "thin_mfma"),
    (48, 8192, 4095, ["bias", "scale"], None, "skinny"),               # 64 rows in turn on a 256-wide step
    (33, 8192, 4097, ["bias", "softmax"], None, "skinny"),             # K = 4160 behind the copies: a 64-wide step
])
def test_ragged_rows_match_the_oracle(dtype, M, N, K, kinds, f32, two_byte):
    prob = inputs.random_problem(81, M, N, K, dtype, kinds)
    call = call_of(prob)
    kernel = f32 if dtype == F32 else two_byte
    check(prob, call, "x,w" if kernel else None)
    text = call.plan()
    if kernel is None:
        return
    family, form = (kernel.split("_") + ["mfma"])[:2]
    assert text.startswith("variant=general+copies:%s_%s_%s" % (family, {F32: "f32", BF16: "bf16", F16: "f16"}[dtype], form)), text
    # no less exact than the general kernel: 2-byte dtypes stage in fp32, fp32 sums at most a quarter of K in one chain
    assert dtype == F32 or "staging=out" not in text, text
    assert dtype != F32 or form == "dot" or int(text.split("split_k=")[1].split()[0]) >= 4, text


@pytest.mark.parametrize("dtype", [F32, BF16])
def test_only_the_operand_that_needs_it_is_copied(dtype):
    prob = inputs.random_problem(83, 1024, 1536, 1024, dtype, ["bias", "relu"])
    check(prob, call_of(prob, x=(1, 0)), "x")
    check(prob, call_of(prob, x=(0, 1)), "x")
    check(prob, call_of(prob, w=(3, 1)), "w")
    check(prob, call_of(prob, x=(1, 0), w=(5, 2)), "x,w")


@pytest.mark.parametrize("dtype,K", [(F32, 1025), (BF16, 1023), (F16, 1028)])
def test_layernorm_of_ragged_rows(dtype, K):
    """The normalised rows are filled up with zeros themselves; only W is copied."""
    prob = inputs.random_problem(85, 1500, 1036, K, dtype, ["bias", "gelu_erf"], ln_pre=True)
    call = call_of(prob, x=(2, 1))
    check(prob, call, "w")
    assert "ln_pre=pass" in call.plan()


@pytest.mark.parametrize("how", ["small", "none", "over_w"])
def test_a_workspace_that_does_not_do_runs_without_copies(how):
    """Nothing that was accepted before the copies existed is refused: the operands are then read as they are."""
    prob = inputs.random_problem(87, 600, 1030, 1001, BF16, ["bias", "relu"])
    call = call_of(prob)
    assert "copies=x,w" in call.plan() and call.workspace_needed >= (600 + 1030) * 1001 * 2
    if how == "small":
        call._p.workspace_bytes = call.workspace_needed - 1
    elif how == "none":
        call._p.workspace, call._p.workspace_bytes = None, 0
    else:
        call._p.workspace = (call._p.w + 255) // 256 * 256
    check(prob, call, None)


def test_static_scratch_runs_without_copies_that_do_not_fit():
    small = inputs.random_problem(89, 600, 1030, 1001, BF16, ["bias"])
    large = inputs.random_problem(89, 600, 8190, 1001, BF16, ["bias"])
    for prob, copies in ((small, True), (large, False)):
        call = call_of(prob)
        assert "copies=x,w" in call.plan()
        got = call.run_static()
        torch.cuda.synchronize()
        assert ("copies" in call.plan()) == copies, call.plan()
        rows = sample_rows(prob.M, 16)
        assert_close(got.cpu()[rows], oracle_rows(prob, rows), BF16, what=call.plan())


@pytest.mark.parametrize("dtype,M,N,K,kinds,copies", [
    (BF16, 600, 1030, 1001, ["bias", "relu"], True), (BF16, 600, 8190, 1001, ["bias", "gelu_erf"], False), (F16, 600, 3001, 2051, ["bias", "layernorm"], False),
    (F32, 4, 1000, 4001, ["bias", "gelu_tanh"], True), (F32, 600, 2049, 1025, ["bias", "residual"], False)])
def test_static_scratch_is_bit_identical_to_a_workspace_of_its_size(dtype, M, N, K, kinds, copies):
    prob = inputs.random_problem(93, M, N, K, dtype, kinds)
    scratch = torch.empty(binding.STATIC_SCRATCH_BYTES, dtype=torch.uint8, device="cuda:0")
    call = call_of(prob, workspace=scratch)
    assert "copies=x,w" in call.plan(), call.plan()
    want = call.run().clone()
    text = call.plan()
    assert ("copies" in text) == copies, text
    call.out.fill_(float("nan"))
    got = call.run_static()
    torch.cuda.synchronize()
    assert call.plan() == text
    assert torch.equal(got.view(torch.uint8), want.view(torch.uint8))


def test_copies_under_capture():
    prob = inputs.random_problem(91, 1000, 1030, 1001, F16, ["bias", "residual", "layernorm"])
    call = call_of(prob)
    want = call.run().clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call.run()
    for _ in range(3):
        call.out.fill_(float("nan"))
        call.workspace.fill_(255)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(call.out, want)
