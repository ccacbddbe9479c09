"""GPU parity of the sum of slabs with a row reduction in the same pass, at the widths where a row takes another wave."""
import pytest
import torch

from paper_2511_16964_amd import inputs

from parity import assert_close, oracle_rows, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("kinds", [["bias", "residual", "layernorm"], ["gelu_tanh", "softmax", "scale"]])
@pytest.mark.parametrize("N", [256, 512, 513, 768, 769, 1536, 1537, 2049, 2304, 2560, 2561, 3071, 4096, 4097, 7680, 7681])
def test_widths_around_a_wave(dtype, kinds, N):
    print("[case] waves of a row", dtype, N, kinds, flush=True)
    prob = inputs.random_problem(147 + N, 6, N, 512, dtype, kinds)
    got, call = run_gpu(prob, "tiled128", poison=True, split=4)
    assert "reduction=one_pass" in call.plan(), call.plan()
    assert_close(got, oracle_rows(prob), dtype, what=call.plan())
