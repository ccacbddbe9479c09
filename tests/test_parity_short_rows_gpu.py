"""GPU parity of the pass behind a row reduction over short rows, at the widths where its forms meet and at every number of partials
that its combine treats differently (1 .. 33 of them)."""
import pytest
import torch

from paper_2511_16964_amd import inputs

from parity import assert_close, oracle_rows, run_gpu

pytestmark = pytest.mark.gpu

F32, BF16, F16 = torch.float32, torch.bfloat16, torch.float16


@pytest.mark.parametrize("N", [1, 8, 15, 16, 17, 64, 65, 130, 257, 272, 504, 511, 512, 513, 520, 528, 1023, 1024, 1025, 1032, 2056])
@pytest.mark.parametrize("dtype,variant,kinds", [
    (BF16, "general", ["bias", "layernorm"]), (F16, "tiled128", ["bias", "residual", "layernorm", "relu"]), (F32, "general", ["layernorm", "bias"]), (F32, "tiled128", ["layernorm"]),
    (BF16, "tiled128", ["softmax"]), (F16, "general", ["bias", "softmax", "scale"]), (F32, "general", ["softmax"]),
])
def test_widths_at_the_edges_of_the_forms(N, dtype, variant, kinds):
    prob = inputs.random_problem(171, 1030 if "softmax" in kinds and N <= 1025 else 37, N, 64, dtype, kinds)   # (softmax: from 1024 rows on)
    print("[case] short rows", dtype, variant, N, kinds, flush=True)
    got, call = run_gpu(prob, variant, split=1, poison=True)
    assert_close(got, oracle_rows(prob), dtype, what=call.plan())
