"""GPU parity of calls with K split and one row reduction: the sum of the slabs, the reduction and the ops behind it in one pass
(reduce_rows) up to 8192 columns, in two behind that; every remainder of a group of four columns and of a batch of slabs."""
import pytest
import torch

from paper_2511_16964_amd import binding, inputs

from parity import assert_close, oracle_rows, run_gpu, sample_rows, to_dev, dev_epilogue

pytestmark = pytest.mark.gpu

F32, BF16, F16 = torch.float32, torch.bfloat16, torch.float16


@pytest.mark.parametrize("dtype", [F32, BF16, F16])
@pytest.mark.parametrize("kinds", [["bias", "residual", "layernorm"], ["gelu_tanh", "softmax", "scale", "residual"], ["bias", "scale", "logsumexp"]])
@pytest.mark.parametrize("N", [1, 3, 4, 5, 255, 257, 1023, 1024, 1025, 2047, 2048, 2050, 8191, 8192, 8193])
def test_every_width(dtype, kinds, N):
    M, K, split = 5, 512, 3 if N % 2 else 8
    prob = inputs.random_problem(141 + N, M, N, K, dtype, kinds)
    print("[case]", dtype, N, kinds, split, flush=True)
    got, call = run_gpu(prob, "tiled128", poison=True, split=split)
    assert "split_k=%d " % split in call.plan(), call.plan()
    assert ("reduction=one_pass" in call.plan()) == (N <= 8192), call.plan()
    assert_close(got, oracle_rows(prob), dtype, what=call.plan())


@pytest.mark.parametrize("split", [2, 4, 5, 7, 8, 9, 15, 16, 17])
@pytest.mark.parametrize("N", [260, 2000, 3001])
def test_every_number_of_slabs(split, N):
    prob = inputs.random_problem(143, 70, N, 64 * 17, BF16, ["bias", "store", "layernorm", "relu"])
    print("[case]", split, N, flush=True)
    x, w, b, ep = to_dev(prob.x), to_dev(prob.w), to_dev(prob.b), dev_epilogue(prob.epilogue)
    store = next(e[1] for e in ep if e[0] == "store")
    store.fill_(float("nan"))
    call = binding.Call(x, w, b, ep, variant="tiled128", split=split)
    got = call.run().cpu()
    assert_close(got, oracle_rows(prob), BF16, what=call.plan())
    plain = inputs.Problem("x", BF16, prob.x, prob.w, prob.b, [("bias",)])
    assert_close(store.cpu(), oracle_rows(plain), BF16, what="store " + call.plan())


def test_residual_behind_the_reduction_in_the_output_itself():
    prob = inputs.random_problem(145, 300, 1000, 1024, F16, ["bias", "softmax", "residual"])
    x, w, b, ep = to_dev(prob.x), to_dev(prob.w), to_dev(prob.b), dev_epilogue(prob.epilogue)
    out = ep[2][1]
    call = binding.Call(x, w, b, ep, out=out, variant="tiled128", split=4)
    assert "staging=workspace_f32" in call.plan(), call.plan()
    got = call.run().cpu()
    rows = sample_rows(300, 24)
    assert_close(got[rows], oracle_rows(prob, rows), F16, what=call.plan())
