"""GPU parity of grouped calls on the 256 tile whose groups end in every height that the last tile row may run at (64, 128, 192 or
256 rows), and of the tile that an automatic plan takes."""
import pytest
import torch

from paper_2511_16964_amd import inputs

from parity import assert_close, oracle_grouped, run_grouped_gpu

pytestmark = pytest.mark.gpu

BF16, F16 = torch.bfloat16, torch.float16
COUNTS = [1, 63, 64, 65, 0, 127, 128, 129, 191, 192, 193, 255, 256, 257, 300, 16, 511, 33]


@pytest.mark.parametrize("dtype,N,K,kinds", [
    (BF16, 512, 64, ["bias", "relu", "residual"]), (F16, 260, 136, ["bias", "scale"]), (BF16, 387, 200, ["bias", "residual"]), (F16, 384, 320, ["residual", "bias"]),
])
def test_groups_end_at_every_height(dtype, N, K, kinds):
    gp = inputs.random_grouped(161, COUNTS, N, K, dtype, kinds, integer=True)   # exact sums
    print("[case] heights", dtype, N, K, kinds, flush=True)
    got, call = run_grouped_gpu(gp, "tiled256")
    assert "tile=256x256" in call.plan(), call.plan()
    assert torch.equal(got.double(), torch.from_numpy(oracle_grouped(gp)).to(dtype).double()), call.plan()


@pytest.mark.parametrize("dtype,kinds", [(BF16, ["bias", "layernorm"]), (F16, ["bias", "gelu_tanh", "residual", "layernorm"]), (BF16, ["softmax"])])
def test_row_reductions_over_every_height(dtype, kinds):
    gp = inputs.random_grouped(163, COUNTS, 392, 192, dtype, kinds)
    print("[case] heights, rows", dtype, kinds, flush=True)
    got, call = run_grouped_gpu(gp, "tiled256")
    assert "tile=256x256" in call.plan(), call.plan()
    assert_close(got, oracle_grouped(gp), dtype, what=call.plan())


@pytest.mark.parametrize("counts,N,K,tile", [([700, 742, 301, 1100, 642, 900, 689, 700], 2496, 1920, 128), ([250] * 32, 2560, 3840, 256)])
def test_the_tile_of_an_automatic_plan(counts, N, K, tile):
    gp = inputs.random_grouped(165, counts, N, K, BF16, ["bias"])
    got, call = run_grouped_gpu(gp)
    assert "tile=%dx%d" % (tile, tile) in call.plan(), call.plan()
    rows = list(range(0, sum(counts), 97))
    assert_close(got[rows], oracle_grouped(gp, rows), BF16, what=call.plan())
