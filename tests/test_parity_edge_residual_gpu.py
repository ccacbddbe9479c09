"""GPU parity of residual operands whose rows lie at any address, in the tiled kernels' epilogue: every remainder of four columns, rows
and columns that end inside a wave's tile, a second residual operand, which is read the other way, and rows of under four columns."""
import pytest
import torch

from paper_2511_16964_amd import inputs

from parity import assert_close, oracle_rows, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", ["tiled128", "tiled256"])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
@pytest.mark.parametrize("M", [1, 33, 129, 300])
@pytest.mark.parametrize("N,kinds", [
    (1, ["bias", "residual"]), (3, ["residual", "relu"]), (5, ["bias", "residual"]), (6, ["residual", "scale"]), (7, ["residual", "residual"]), (63, ["bias", "residual"]),
    (129, ["residual", "bias"]), (130, ["bias", "relu", "residual", "residual"]), (131, ["residual", "layernorm"]), (257, ["bias", "residual", "softmax"]), (515, ["scale", "residual"]),
])
def test_any_width(variant, dtype, M, N, kinds):
    prob = inputs.random_problem(161 + N, M, N, 192, dtype, kinds, integer="layernorm" not in kinds and "softmax" not in kinds)
    print("[case] edge residual", variant, dtype, M, N, kinds, flush=True)
    got, call = run_gpu(prob, variant, poison=True)
    assert "edge" in call.plan(), call.plan()
    assert_close(got, oracle_rows(prob), dtype, what=call.plan())
