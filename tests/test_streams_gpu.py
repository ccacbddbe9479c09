"""Calls that run on another stream than the one their scratch memory was allocated under: the memory must not be handed out
again while that stream still uses it, also when the call object is gone."""
import pytest
import torch

from paper_2511_16964_amd import binding

pytestmark = pytest.mark.gpu

BF16 = torch.bfloat16


def rand(*shape):
    return torch.rand(shape, device="cuda:0").to(BF16) - 0.5


def ragged_linear():
    return binding.Call(rand(1024, 1001), rand(1030, 1001), rand(1030), [("bias",)])


def layernorm():
    return binding.Call(rand(4096, 512), rand(8192, 512), None, [("layernorm", None, None, 1e-5)])


def decode_attention():
    return binding.AttentionCall(rand(4, 1, 16, 128), rand(4, 8192, 16, 128), rand(4, 8192, 16, 128), 1)


def block():
    return binding.AttentionBlockCall(rand(2, 512, 512), rand(1536, 512), None, rand(512, 512), None, 8, True)


@pytest.mark.parametrize("make", [ragged_linear, layernorm, decode_attention, block])
@pytest.mark.parametrize("how", ["argument", "current"])
def test_scratch_memory_is_held_until_the_stream_is_through(make, how):
    want = make().run().float().norm()
    call, side = make(), torch.cuda.Stream()
    operands = list(call._tensors if hasattr(call, "_tensors") else call._keep)   # (the caller's, who keeps them)
    memory = operands.pop() if make is block else call.workspace
    start, size = memory.data_ptr(), memory.numel()
    del memory
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(200_000_000)   # some 0.1 s of waiting ahead of the call
        if how == "current":
            out = call.run()
    if how == "argument":
        out = call.run(side)
    del call
    held = not side.query()
    taken = [torch.empty(n, dtype=torch.uint8, device="cuda:0").fill_(255) for n in (size, size // 2, size // 4)]
    assert held, "the call was over before the memory could be asked for again"
    for t in taken:
        assert t.data_ptr() + t.numel() <= start or start + size <= t.data_ptr()
    side.synchronize()
    assert torch.isfinite(out.float()).all() and torch.isfinite(want)
