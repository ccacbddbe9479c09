"""GPU parity of a LayerNorm of x over K in front of the multiplication (normalisation -> projection): inside the
dot-product kernel's own sweep for a few rows of x, as a pass into the workspace in front of every other kernel.  The
oracle normalises the stored x in float64 (definition pinned on the CPU side) and multiplies the unrounded result."""
import numpy as np
import pytest
import torch

from paper_2511_16964_amd import binding, inputs

from parity import assert_close, oracle_rows, run_gpu, sample_rows

pytestmark = pytest.mark.gpu

F32, BF16, F16 = torch.float32, torch.bfloat16, torch.float16


def announce(*a):
    print("[case]", *a, flush=True)


@pytest.mark.parametrize("dtype,M", [(BF16, 1), (BF16, 2), (BF16, 3), (BF16, 4), (F16, 1), (F16, 4), (F32, 1), (F32, 3), (F32, 4)])
@pytest.mark.parametrize("N,K", [(1024, 1024), (4096, 4096), (520, 2048), (4100, 4104)])
@pytest.mark.parametrize("kinds", [["bias", "gelu_erf"], ["bias", "relu", "layernorm"]])
def test_few_rows_normalise_inside_the_dot_product_kernel(dtype, M, N, K, kinds):
    prob = inputs.random_problem(61, M, N, K, dtype, kinds, ln_pre=True)
    announce("ln_pre fused", dtype, M, N, K, kinds)
    got, call = run_gpu(prob, "thin", poison=True)
    assert "ln_pre=fused" in call.plan() and "_dot" in call.plan(), call.plan()
    assert_close(got, oracle_rows(prob), dtype, what="ln_pre fused %s" % call.plan())


@pytest.mark.parametrize("dtype", [BF16, F32])
def test_fused_form_without_gamma_or_beta_and_off_centre_rows(dtype):
    """gamma / beta absent (1 / 0), and rows whose mean is 30 deviations from zero (the kernel's one-sweep variance
    is E[x^2] - mean^2 in fp32)."""
    for g_on, b_on, x_mean in ((False, True, 0.5), (True, False, 0.5), (False, False, 0.5), (True, True, 30.0)):
        prob = inputs.random_problem(63, 2, 2048, 4096, dtype, ["bias"], ln_pre=True, x_mean=x_mean)
        e = prob.epilogue[0]
        prob.epilogue[0] = ("layernorm_pre", e[1] if g_on else None, e[2] if b_on else None, e[3])
        announce("ln_pre fused", dtype, g_on, b_on, x_mean)
        got, call = run_gpu(prob, "thin", poison=True)
        assert "ln_pre=fused" in call.plan()
        assert_close(got, oracle_rows(prob), dtype, what="ln_pre fused gamma %s beta %s mean %s" % (g_on, b_on, x_mean))


@pytest.mark.parametrize("dtype,M,N,K", [   # the longest rows that are normalised into LDS, and the shortest that are not
    (BF16, 1, 4097, 16384), (BF16, 1, 4096, 16392), (F32, 1, 4096, 8192), (F32, 1, 4099, 8196),     # 16 waves, a row of W each
    (F16, 1, 1000, 8192), (F16, 1, 1001, 8200), (F32, 2, 1024, 4096), (F32, 2, 1024, 4100), (BF16, 2, 520, 8192), (BF16, 2, 516, 8200),
    (BF16, 1, 17, 8), (F32, 2, 5, 4), (F16, 2, 33, 520), (BF16, 1, 4096, 2056),                      # one vector, part of a block
])
@pytest.mark.parametrize("x_mean", [0.5, 300.0])
def test_one_and_two_rows_at_the_limits(dtype, M, N, K, x_mean):
    """A mean of hundreds of deviations: the form that holds x takes the deviations from the mean itself (the sums of the
    other, which take longer rows, are good to a mean of 30)."""
    held = K <= (16384 if M == 1 and N >= 4096 and K >= 2048 else 8192) // (2 if dtype == F32 else 1)
    if dtype != F32:   # (x itself is rounded to the dtype: keep its deviations)
        x_mean = min(x_mean, 30.0)
    if not held:
        x_mean = min(x_mean, 30.0)
    prob = inputs.random_problem(71, M, N, K, dtype, ["bias"], ln_pre=True, x_mean=x_mean)
    announce("ln_pre held", dtype, M, N, K, x_mean)
    got, call = run_gpu(prob, "thin", poison=True)
    assert "ln_pre=fused" in call.plan(), call.plan()
    assert_close(got, oracle_rows(prob), dtype, what="ln_pre held %s" % call.plan())


@pytest.mark.parametrize("dtype,variant,M,N,K", [
    (BF16, "auto", 300, 520, 512), (BF16, "tiled256", 513, 772, 1024), (BF16, "tiled128", 77, 132, 128), (BF16, "skinny256", 64, 4096, 1024),
    (BF16, "thin", 16, 1024, 2048), (BF16, "general", 33, 70, 100), (F16, "auto", 130, 260, 200), (F32, "auto", 130, 260, 203),
    (F32, "tiled128", 200, 264, 512), (BF16, "auto", 1000, 132, 147), (BF16, "auto", 2, 64, 64), (F32, "thin", 8, 4096, 4096), (F32, "thin", 5, 1024, 2048),
])
@pytest.mark.parametrize("kinds", [["bias", "gelu_tanh"], ["bias", "residual", "layernorm"], ["scale", "softmax"]])
def test_other_shapes_normalise_in_a_pass_of_their_own(dtype, variant, M, N, K, kinds):
    prob = inputs.random_problem(67, M, N, K, dtype, kinds, ln_pre=True)
    announce("ln_pre pass", dtype, variant, M, N, K, kinds)
    got, call = run_gpu(prob, variant, poison=True)
    assert "ln_pre=pass" in call.plan(), call.plan()
    assert_close(got, oracle_rows(prob), dtype, what="ln_pre pass %s" % call.plan())


@pytest.mark.parametrize("dtype", [F32, BF16, F16])
@pytest.mark.parametrize("M,N,K", [(1, 4100, 2056), (1, 520, 1160), (2, 520, 1160), (2, 520, 8)])   # rows that are no whole KB
@pytest.mark.parametrize("which", ["gamma", "beta"])
def test_an_infinite_gamma_or_beta_reaches_the_result(dtype, M, N, K, which):
    """One infinite element of the affine part makes every output that its weight does not cancel infinite, none NaN."""
    prob = inputs.random_problem(72, M, N, K, dtype, [], ln_pre=True)
    for at in (0, K - 1):
        ep = [tuple(t.clone() if isinstance(t, torch.Tensor) else t for t in e) for e in prob.epilogue]
        ep[0][1 if which == "gamma" else 2][at] = float("inf")
        w = prob.w.clone()
        w[:, at] = torch.tensor([1.0, -1.0]).repeat(N)[:N].to(dtype)
        p = inputs.Problem("x", dtype, prob.x, w, prob.b, ep)
        announce("ln_pre infinite", dtype, M, N, K, which, at)
        got, call = run_gpu(p, "thin", poison=True)
        assert "ln_pre=fused" in call.plan(), call.plan()
        x = prob.x.double()
        sign = torch.ones(M) if which == "beta" else torch.sign(x[:, at] - x.mean(1))
        want = torch.sign(w[:, at].double())[None] * sign[:, None].double() * float("inf")
        assert torch.equal(got.double(), want), (call.plan(), at)


def test_misaligned_x_rows_still_reach_the_fast_kernels():
    """The normalised copy is contiguous and aligned whatever x looks like: x with an odd leading dimension and a
    2-byte offset takes the tiled kernel after the pass (alone it would fall to the general kernel)."""
    prob = inputs.random_problem(69, 1024, 1024, 1024, BF16, ["bias", "relu"], ln_pre=True)
    dev = "cuda:0"
    buf = torch.zeros(1024, 1024 + 3, dtype=BF16, device=dev)
    xv = buf[:, 1:1025]
    xv.copy_(prob.x.to(dev))
    ep = [tuple(t.to(dev) if isinstance(t, torch.Tensor) else t for t in e) for e in prob.epilogue]
    call = binding.Call(xv, prob.w.to(dev), prob.b.to(dev), ep)
    got = call.run().cpu()
    assert "tiled" in call.plan() and "ln_pre=pass" in call.plan(), call.plan()
    assert_close(got, oracle_rows(prob), BF16, what="misaligned x")
    plain = binding.Call(xv, prob.w.to(dev), prob.b.to(dev), ep[1:])
    assert "general" in plain.plan()


def test_full_size_projection_behind_a_layernorm():
    """A transformer block's normalisation -> projection at benchmark size (4096 tokens, 4096 -> 4096), sampled rows."""
    prob = inputs.random_problem(71, 4096, 4096, 4096, BF16, ["bias", "gelu_erf"], ln_pre=True)
    announce("ln_pre full size")
    got, call = run_gpu(prob, poison=True)
    assert "ln_pre=pass" in call.plan() and "tile=256x256" in call.plan()
    assert torch.isfinite(got.float()).all()
    rows = sample_rows(4096, 32)
    assert_close(got[rows], oracle_rows(prob, rows), BF16, what="ln_pre full size")
