"""GPU parity of attention over heads of 256: one to five key blocks (the loop takes two at a time), and rows whose largest score
grows from block to block, so that the sums held in accumulation registers are scaled between the blocks."""
import pytest
import torch

from paper_2511_16964_amd import binding, inputs

from parity import assert_close, attention_reference

pytestmark = pytest.mark.gpu

BF16, F16 = torch.bfloat16, torch.float16


@pytest.mark.parametrize("dtype", [BF16, F16])
@pytest.mark.parametrize("causal", [0, 1, 48])
@pytest.mark.parametrize("growth", [0.0, 0.5])
@pytest.mark.parametrize("T,Tk", [(33, 33), (64, 64), (129, 129), (40, 192), (192, 192), (257, 257), (100, 320)])
def test_heads_of_256(dtype, causal, growth, T, Tk):
    print("[case] attention 256", dtype, causal, growth, T, Tk, flush=True)
    q = inputs.make_qkv(600 + T, 2, T, 3, 256, dtype)[:, :, 0]
    kv = inputs.make_qkv(700 + Tk, 2, Tk, 3, 256, dtype)
    k, v = kv[:, :, 1], kv[:, :, 2]
    if growth:  # keys of block j point along the head's own query direction, longer with j: every block's maximum is 2^8 and more above the last one's
        block = torch.arange(Tk).div(64, rounding_mode="floor").float()
        mean = q.float().mean(1, keepdim=True)
        q = (q.float() * 0.25 + 4.0 * mean / mean.norm(dim=-1, keepdim=True)).to(dtype)
        k = (k.float() * 0.25 + (block * growth * 64.0).view(1, -1, 1, 1) * mean / mean.norm(dim=-1, keepdim=True)).to(dtype)
    got = binding.attention(q.to("cuda:0"), k.to("cuda:0"), v.to("cuda:0"), causal)
    torch.cuda.synchronize()
    f = inputs.to_f64
    ref, extra = attention_reference(f(q), f(k), f(v), causal, dtype)
    assert_close(got.cpu(), ref, dtype, extra=extra)
