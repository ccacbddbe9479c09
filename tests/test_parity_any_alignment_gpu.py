"""GPU parity of epilogues and row passes over rows that start at any element: vector accesses at unaligned addresses for
whole groups of columns, the columns behind them one by one."""
import pytest
import torch

from paper_2511_16964_amd import binding, inputs

from parity import assert_close, oracle_rows, sample_rows, to_dev

pytestmark = pytest.mark.gpu

F32, BF16, F16 = torch.float32, torch.bfloat16, torch.float16
GUARD = 7.0


def shifted(t, pad, shift):
    """t at a start `shift` elements into a buffer of GUARD, rows `pad` elements longer: (buffer, view)."""
    rows, cols = (1, t.numel()) if t.dim() == 1 else t.shape
    buf = torch.full((rows * (cols + pad) + shift + 16,), GUARD, dtype=t.dtype, device="cuda:0")
    view = buf[shift:shift + rows * (cols + pad)].view(rows, cols + pad)[:, :cols]
    view.copy_(t.reshape(rows, cols).to("cuda:0"))
    return buf, (view[0] if t.dim() == 1 else view)


@pytest.mark.parametrize("dtype", [F32, BF16, F16])
@pytest.mark.parametrize("N", [3, 7, 8, 9, 127, 130, 2047, 2048, 2049, 2055, 2056, 2057])
@pytest.mark.parametrize("kinds,variant", [(["bias", "residual", "layernorm"], "tiled128"), (["softmax", "residual"], "tiled256"),
                                           (["residual", "layernorm", "relu"], "split"), (["bias", "residual", "gelu_tanh"], "tiled128")])
def test_rows_at_any_element(dtype, N, kinds, variant):
    M, K = (300, 128) if variant != "split" else (130, 512)
    prob = inputs.random_problem(95 + N, M, N, K, dtype, kinds)
    print("[case]", dtype, N, kinds, variant, flush=True)
    ep, keep = [], []
    for e in prob.epilogue:
        if e[0] in ("residual", "layernorm"):
            moved = [shifted(t, 3, 1) if isinstance(t, torch.Tensor) else (None, t) for t in e[1:]]
            keep += moved
            e = (e[0],) + tuple(v for _, v in moved)
        ep.append(e)
    buf, out = shifted(torch.full((M, N), float("nan"), dtype=dtype), 5, 3)
    b = shifted(prob.b, 0, 1)[1] if prob.b is not None else None
    how = dict(variant="tiled128", split=2) if variant == "split" else dict(variant=variant)
    call = binding.Call(to_dev(prob.x), to_dev(prob.w), b, ep, out=out, **how)
    got = call.run().cpu()
    torch.cuda.synchronize()
    rows = sample_rows(M, 24, tile=64)
    assert_close(got[rows], oracle_rows(prob, rows), dtype, what=call.plan())
    # nothing outside the rows was written
    mask = torch.ones_like(buf, dtype=torch.bool)
    mask[3:3 + M * (N + 5)].view(M, N + 5)[:, :N] = False
    assert (buf[mask] == GUARD).all(), call.plan()
