"""GPU parity of the order in which tiles are walked: blocks of 6 tile rows in a matrix of many tile columns (a last block of
fewer rows, a last tile column of one element), blocks of a group's own in the grouped form (fewer, as many and more tile
rows than a block holds).  Small integers make every value exact: a tile computed twice, not at all or in another's place
shows as a whole number, or as the NaN that the output is filled with."""
import numpy as np
import pytest
import torch

from paper_2511_16964_amd import binding, inputs

from parity import oracle_grouped, oracle_rows, run_gpu, run_grouped_gpu

pytestmark = pytest.mark.gpu

BF16, F8 = torch.bfloat16, torch.float8_e4m3fn


@pytest.mark.parametrize("dtype,M,N,K", [
    (BF16, 256 * 8 + 1, 256 * 32, 64),       # 9 x 32 tiles: blocks of 6 and 3
    (BF16, 256 * 13, 256 * 31 + 1, 32),      # 13 x 32: a last block of one row, a last column of one element
    (F8, 256 * 12 - 3, 256 * 33 - 4, 32),    # 12 x 33: whole blocks, ids that 8 does not divide
    (BF16, 256 * 8, 256 * 32, 64),           # 256 tiles: blocks of 4
    (BF16, 256 * 9, 256 * 31, 64),           # 31 tile columns: blocks of 4
])
def test_every_tile_of_a_wide_matrix_is_computed(dtype, M, N, K):
    prob = inputs.random_problem(301, M, N, K, dtype, ["bias", "relu"], integer=True)
    print("[case]", dtype, M, N, K, flush=True)
    got, call = run_gpu(prob, "tiled256", poison=True)
    assert "tile=256x256" in call.plan(), call.plan()
    assert np.array_equal(got.to(torch.float64).numpy(), oracle_rows(prob)), call.plan()


@pytest.mark.parametrize("variant,tile", [("tiled128", 128), ("tiled256", 256)])
@pytest.mark.parametrize("tile_rows", [[8, 9], [1, 7, 17, 0, 3], [16, 2, 25]])
def test_every_tile_of_the_groups_is_computed(variant, tile, tile_rows):
    counts = [max(0, n * tile - 5 * i) for i, n in enumerate(tile_rows)]
    gp = inputs.random_grouped(302, counts, 3 * tile + 4, 64, BF16, ["bias", "relu"], integer=True)
    print("[case]", variant, counts, flush=True)
    got, call = run_grouped_gpu(gp, variant)
    assert np.array_equal(got.to(torch.float64).numpy(), oracle_grouped(gp)), call.plan()
