"""GPU parity of attention over heads of 256: one to five key blocks (the loop takes two at a time), and rows whose largest score
grows from block to block, so that the sums held in accumulation registers are scaled between the blocks."""
import numpy as np
import pytest
import torch

import oracle
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


@pytest.mark.parametrize("dtype", [BF16, F16])
@pytest.mark.parametrize("causal", [0, 1, 48])
@pytest.mark.parametrize("block", [1, 2, 3, 4])
@pytest.mark.parametrize("T,Tk", [(33, 320), (130, 320), (257, 321)])
def test_scaled_sums_are_a_visible_share(dtype, causal, block, T, Tk):
    """One key, the first of a block, scores 2^8.6 above every other: the reference moves by that much there (it does from 2^8 on), and the
    64 to 256 keys in front of it keep 64 / (64 + 388) to 256 / (256 + 388) of the weight.  Sums that were cleared instead of scaled
    would leave the criterion, as would sums left as they are."""
    print("[case] attention 256 scaled", dtype, causal, block, T, Tk, flush=True)
    D, H, B = 256, 3, 2
    rng = np.random.default_rng(900 + 10 * block + T)
    u = rng.standard_normal((1, 1, H, D))
    u /= np.linalg.norm(u, axis=-1, keepdims=True)
    q = 16.0 * u + 0.02 * rng.standard_normal((B, T, H, D))
    k = rng.standard_normal((B, Tk, H, D))
    k -= (k * u).sum(-1, keepdims=True) * u
    key = 64 * block
    k[:, key] += 8.6 * np.log(2.0) * u[0]                    # 16 / sqrt(256) = 1
    v = rng.standard_normal((B, Tk, H, D)) + np.where(np.arange(Tk) < key, 1.0, -1.0)[None, :, None, None]
    q, k, v = (torch.from_numpy(t).to(dtype) for t in (q, k, v))
    f = inputs.to_f64
    limit = np.full(T, Tk) if causal == 0 else np.minimum(Tk, ((np.arange(T) + Tk - T) // causal + 1) * causal)
    sees = limit > key
    scores = np.einsum("bthd,bjhd->bhtj", f(q), f(k)) / 16.0 / np.log(2.0)
    rise = scores[..., key] - scores[..., :key].max(-1)
    assert rise.min() > 8.2 and rise.max() < 9.2, (rise.min(), rise.max())    # the reference moves, by little more than it must
    ref, extra = attention_reference(f(q), f(k), f(v), causal, dtype)
    if sees.any():
        w = np.where(np.arange(Tk) < limit[sees][:, None], 2.0 ** (scores - scores[..., key:key + 1])[:, :, sees], 0.0)
        for factor in (0.0, 2.0 ** 8.6):                        # cleared, not scaled
            wrong = np.where(np.arange(Tk) < key, factor, 1.0) * w
            bad = np.einsum("bhtj,bjhd->bthd", wrong / wrong.sum(-1, keepdims=True), f(v))
            with pytest.raises(AssertionError):
                assert_close(torch.from_numpy(bad), ref[:, sees], dtype, extra=extra[:, sees])
    got = binding.attention(q.to("cuda:0"), k.to("cuda:0"), v.to("cuda:0"), causal)
    torch.cuda.synchronize()
    assert_close(got.cpu(), ref, dtype, extra=extra)
