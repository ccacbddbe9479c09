"""GPU parity of attention with a few new queries per sequence (T <= 32): the kernel whose waves share out the keys, in
one range and cut into several that a second kernel puts together.  Same oracle and criterion as the other attention tests."""
import pytest
import torch

from paper_2511_16964_amd import binding, inputs

from parity import assert_close, attention_reference

pytestmark = pytest.mark.gpu

BF16, F16 = torch.bfloat16, torch.float16
DEV = "cuda:0"


@pytest.mark.parametrize("dtype,B,H,D,T,Tk,causal,ranges", [
    # one range: fewer blocks of 32 keys than waves, exactly as many, one more; the tile's last and first query count
    (BF16, 2, 3, 128, 1, 1, 1, False), (F16, 2, 3, 64, 32, 32, 1, False), (BF16, 1, 5, 32, 31, 33, 0, False),
    (BF16, 2, 3, 128, 2, 128, 1, False), (F16, 2, 3, 128, 5, 129, 1, False), (BF16, 2, 3, 256, 3, 65, 0, False),
    (BF16, 40, 16, 64, 1, 97, 1, False), (BF16, 2, 2, 128, 1, 31, 7, False),
    # several ranges: whole and ragged last blocks, more ranges than lanes of one group reading them back, masks that end
    # inside the last range or (groups of tokens) leave whole blocks of it to some queries only
    (BF16, 1, 1, 128, 1, 8192, 1, True), (F16, 2, 3, 128, 2, 4097, 1, True), (BF16, 1, 2, 64, 32, 3000, 1, True),
    (F16, 1, 2, 32, 17, 5001, 0, True), (BF16, 1, 3, 256, 5, 2047, 1, True), (BF16, 1, 2, 64, 30, 2000, 16, True),
    (BF16, 1, 1, 32, 32, 1100, 1100, True), (F16, 3, 25, 128, 1, 2500, 1, True),
])
def test_few_queries_against_many_keys(dtype, B, H, D, T, Tk, causal, ranges):
    print("[case] attention decode", dtype, B, H, D, T, Tk, causal, flush=True)
    q = inputs.make_qkv(40 + T, B, T, H, D, dtype)[:, :, 0]
    kv = inputs.make_qkv(41 + Tk, B, Tk, H, D, dtype)
    f = inputs.to_f64
    ref, extra = attention_reference(f(q), f(kv[:, :, 1]), f(kv[:, :, 2]), causal, dtype)
    dkv = kv.to(DEV)
    call = binding.AttentionCall(q.to(DEV), dkv[:, :, 1], dkv[:, :, 2], causal)
    assert (call.workspace is not None) == ranges
    if ranges:
        call.workspace.fill_(255)   # NaNs: every value the second kernel reads has been written
    for _ in range(2):
        call.out.zero_()
        call.run()
        torch.cuda.synchronize()
        assert_close(call.out.cpu(), ref, dtype, extra=extra)
    # without a workspace: one range
    out = torch.zeros_like(call.out)
    call._p.o = out.data_ptr()
    assert binding.lib().fle_attention_run(call._pref) == 0
    torch.cuda.synchronize()
    assert_close(out.cpu(), ref, dtype, extra=extra)


@pytest.mark.parametrize("dtype,B,H,D,T,Tk,causal", [
    # the fewest keys that take the kernel whose waves share them out: fewer blocks of 32 than waves, ragged last blocks
    (BF16, 80, 16, 32, 1, 1, 1), (F16, 49, 16, 32, 5, 33, 1), (BF16, 49, 16, 32, 32, 97, 32), (F16, 4, 16, 32, 3, 257, 1),
    (BF16, 2, 8, 64, 32, 513, 1), (F16, 3, 5, 64, 1, 512, 0), (BF16, 24, 8, 128, 7, 529, 1), (F16, 12, 16, 128, 32, 512, 1),
    (BF16, 2, 3, 256, 1, 1, 1), (F16, 1, 5, 256, 8, 31, 1), (BF16, 17, 16, 256, 32, 65, 1), (F16, 33, 8, 256, 9, 32, 0),
])
def test_sharing_out_the_fewest_keys(dtype, B, H, D, T, Tk, causal):
    print("[case] attention decode, few keys", dtype, B, H, D, T, Tk, causal, flush=True)
    q = inputs.make_qkv(50 + T, B, T, H, D, dtype)[:, :, 0]
    kv = inputs.make_qkv(51 + Tk, B, Tk, H, D, dtype)
    f = inputs.to_f64
    ref, extra = attention_reference(f(q), f(kv[:, :, 1]), f(kv[:, :, 2]), causal, dtype)
    dkv = kv.to(DEV)
    call = binding.AttentionCall(q.to(DEV), dkv[:, :, 1], dkv[:, :, 2], causal)
    call.out.fill_(float("nan"))
    call.run()
    torch.cuda.synchronize()
    assert call.plan().startswith("variant=decode_attention_%s D=%d queries=32 ranges=1 " % ("f16" if dtype == F16 else "bf16", D)), call.plan()
    assert_close(call.out.cpu(), ref, dtype, extra=extra)


def test_ranges_that_one_query_cannot_see_and_large_scores():
    """32 queries under a group mask over scores of a hundred and more: reference points far apart between the ranges."""
    B, H, D, T, Tk, G = 1, 2, 128, 32, 2048, 32
    q, kv = inputs.make_qkv(5, B, T, H, D, BF16, spread=3.0)[:, :, 0], inputs.make_qkv(6, B, Tk, H, D, BF16, spread=3.0)
    f = inputs.to_f64
    ref, extra = attention_reference(f(q), f(kv[:, :, 1]), f(kv[:, :, 2]), G, BF16)
    d = kv.to(DEV)
    out = binding.attention(q.to(DEV), d[:, :, 1], d[:, :, 2], G)
    torch.cuda.synchronize()
    assert_close(out.cpu(), ref, BF16, extra=extra)


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("D", [64, 128])
def test_values_that_are_not_finite_reach_the_result_from_every_range(D, bad):
    """A key whose weight underflows to zero still carries a NaN or infinity in its V into the sum (0 x it is NaN), whether
    its range is put together with others or not; the other elements of the head are untouched."""
    B, H, T, Tk = 1, 2, 1, 8192
    q, kv = torch.zeros(B, T, H, D, dtype=BF16), inputs.make_qkv(9, B, Tk, H, D, BF16).clone()
    q[..., 0] = 64.0
    kv[:, :, 1] = 0.0
    kv[:, 0, 1, :, 0] = 64.0     # scores: 64 * 64 / sqrt(D) for the first key, 0 for the others
    kv[0, 5000, 2, 1, 3] = bad   # V of a key far behind it
    d = kv.to(DEV)
    call = binding.AttentionCall(q.to(DEV), d[:, :, 1], d[:, :, 2], 1)
    assert call.workspace is not None
    got = call.run().clone()
    one = torch.zeros_like(got)
    call._p.o = one.data_ptr()
    assert binding.lib().fle_attention_run(call._pref) == 0
    torch.cuda.synchronize()
    for out in (got, one):
        is_nan = torch.isnan(out)
        assert is_nan[0, 0, 1, 3] and int(is_nan.sum()) == 1, out
    assert torch.equal(got.nan_to_num(7.0), one.nan_to_num(7.0))
