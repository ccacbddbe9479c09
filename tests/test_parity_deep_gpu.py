"""GPU parity of the 128 tile with four K steps in LDS: every count of K steps
around the depth of the pipeline, a last step of few chunks, tiles that end inside the matrix, K split, and the calls that the
planner gives to it."""
import pytest
import torch

from paper_2511_16964_amd import binding, inputs

from parity import assert_close, oracle_grouped, oracle_rows, run_gpu, run_grouped_gpu, sample_rows

pytestmark = pytest.mark.gpu

BF16, F16, F8 = torch.bfloat16, torch.float16, torch.float8_e4m3fn
DEEP = 10


def forced(prob, split):
    L = binding.lib()
    L.fle_force_variant(DEEP)
    L.fle_force_split(split)
    try:
        got, call = run_gpu(prob, poison=True)
        assert "+deep" in call.plan(), call.plan()
        return got, call.plan()
    finally:
        L.fle_force_variant(0)
        L.fle_force_split(0)


@pytest.mark.parametrize("dtype,mx", [(BF16, False), (F16, False), (F8, False), (F8, True)])
@pytest.mark.parametrize("steps,chunks", [(1, 8), (1, 1), (2, 8), (3, 1), (4, 8), (5, 7), (6, 8), (9, 3)])   # chunks of 16 bytes in the last step
@pytest.mark.parametrize("M,N,kinds", [(1, 4, ["bias"]), (129, 260, ["bias", "relu", "scale", "residual"]), (300, 131, ["bias", "residual", "layernorm"])])
def test_every_number_of_steps(dtype, mx, steps, chunks, M, N, kinds):
    if mx and chunks != 8:
        pytest.skip("block scales need whole K steps")
    per = 16 if dtype == F8 else 8
    K = (8 * (steps - 1) + chunks) * per
    integer = "layernorm" not in kinds   # sums exact in fp32: any misplaced K step shows as a whole number
    prob = inputs.random_problem(131, M, N, K, dtype, kinds, integer=integer, mx=mx)
    print("[case]", dtype, mx, M, N, K, flush=True)
    got, text = forced(prob, 1)
    assert_close(got, oracle_rows(prob), dtype, what=text)


# Block-scaled operands take whole K steps only: the step counts that the list above gives a partial last step, and no residual in
# front of the counted waits (a staged one makes the first of them stricter).  Five steps are the count whose waits once fell short.
@pytest.mark.parametrize("steps", [3, 5, 7, 8, 9])
@pytest.mark.parametrize("M,N,kinds", [(1, 4, ["bias"]), (129, 260, ["bias", "relu", "scale"]), (300, 131, ["bias"]), (257, 516, ["bias", "residual"])])
def test_block_scales_over_every_number_of_steps(steps, M, N, kinds):
    prob = inputs.random_problem(137, M, N, 128 * steps, F8, kinds, integer=True, mx=True)
    print("[case]", M, N, steps, flush=True)
    got, text = forced(prob, 1)
    assert "_f8mx_" in text, text
    assert torch.equal(got, torch.from_numpy(oracle_rows(prob)).to(BF16)), text   # (exact sums, rounded once)


@pytest.mark.parametrize("M,N,steps,split", [(1024, 4096, 5, 1), (256, 1024, 10, 2), (512, 1024, 15, 3)])   # one range of five steps, and more of them
def test_block_scales_in_ranges_of_five_steps(M, N, steps, split):
    prob = inputs.random_problem(139, M, N, 128 * steps, F8, ["bias", "relu"], integer=True, mx=True)
    print("[case]", M, N, steps, split, flush=True)
    got, text = forced(prob, split)
    assert "_f8mx_" in text and "split_k=%d " % split in text, text
    rows = sample_rows(M, 48, tile=128)
    assert torch.equal(got[rows], torch.from_numpy(oracle_rows(prob, rows)).to(BF16)), text
    assert torch.isfinite(got.float()).all(), text


@pytest.mark.parametrize("dtype", [BF16, F8])
@pytest.mark.parametrize("split", [2, 3, 5])
def test_split_of_k(dtype, split):
    prob = inputs.random_problem(133, 257, 388, 64 * 11 + 16, dtype, ["bias", "gelu_erf", "residual", "layernorm"])
    print("[case]", dtype, split, flush=True)
    got, text = forced(prob, split)
    assert "split_k=%d" % split in text, text
    assert_close(got, oracle_rows(prob), dtype, what=text)


@pytest.mark.parametrize("dtype", [BF16, F16, F8])
@pytest.mark.parametrize("M,N,K,kinds", [
    (1024, 4096, 1024, ["bias", "relu", "residual"]),                # one workgroup per CU, no split
    (640, 1000, 2048, ["bias", "gelu_tanh", "layernorm"]),           # K split
])
def test_automatic_plans(dtype, M, N, K, kinds):
    prob = inputs.random_problem(135, M, N, K, dtype, kinds)
    print("[case]", dtype, M, N, K, flush=True)
    got, call = run_gpu(prob, poison=True)
    assert "+deep" in call.plan(), call.plan()
    rows = sample_rows(M, 32)
    assert torch.isfinite(got.float()).all(), call.plan()
    assert_close(got[rows], oracle_rows(prob, rows), dtype, what=call.plan())


@pytest.mark.parametrize("dtype", [BF16, F16, F8])
@pytest.mark.parametrize("counts,N,K", [
    ([300, 0, 129, 595], 1920, 128 * 5),       # tiles that end inside their group
    ([1, 255, 128, 900], 2047, 128 * 9 + 16),  # rows of out that are not aligned, a last step of one or two chunks
])
def test_automatic_plans_of_grouped_calls(dtype, counts, N, K):
    gp = inputs.random_grouped(141, counts, N, K, dtype, ["bias", "relu"], integer=True)
    print("[case]", dtype, counts, N, K, flush=True)
    got, call = run_grouped_gpu(gp)
    assert "grouped_tiled" in call.plan() and "+deep" in call.plan(), call.plan()
    rows = sample_rows(sum(counts), 64, tile=32)
    assert torch.equal(got[rows].double(), torch.from_numpy(oracle_grouped(gp, rows)).to(got.dtype).double()), call.plan()
