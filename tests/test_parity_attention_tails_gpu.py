"""GPU parity of attention whose last key block holds few keys: the second half of it lies behind some or all queries' limits."""
import pytest
import torch

from paper_2511_16964_amd import binding, inputs

from parity import assert_close, attention_reference

pytestmark = pytest.mark.gpu

BF16, F16 = torch.bfloat16, torch.float16


@pytest.mark.parametrize("dtype", [BF16, F16])
@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("causal", [0, 1, 48])
@pytest.mark.parametrize("T,Tk", [(1, 33), (65, 65), (95, 95), (96, 96), (97, 97), (197, 197), (40, 225), (160, 161), (130, 192)])
def test_last_block_of_few_keys(dtype, D, causal, T, Tk):
    print("[case] attention tail", dtype, D, causal, T, Tk, flush=True)
    q = inputs.make_qkv(400 + T, 2, T, 3, D, dtype)[:, :, 0]
    kv = inputs.make_qkv(500 + Tk, 2, Tk, 3, D, dtype)
    got = binding.attention(q.to("cuda:0"), kv[:, :, 1].to("cuda:0"), kv[:, :, 2].to("cuda:0"), causal)
    torch.cuda.synchronize()
    f = inputs.to_f64
    ref, extra = attention_reference(f(q), f(kv[:, :, 1]), f(kv[:, :, 2]), causal, dtype)
    assert_close(got.cpu(), ref, dtype, extra=extra)
