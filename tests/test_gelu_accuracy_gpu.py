"""GELU-erf on the GPU against float64, value by value: fp32 problems with W = 1 hand x to the epilogue unchanged."""
import pytest
import torch

from paper_2511_16964_amd import fused_linear_epilogue

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24


@pytest.mark.parametrize("M", [8, 128, 2048])   # dot-product, general and tiled kernel
def test_gelu_erf_is_the_float64_value_to_its_stated_error(M):
    """|error| <= 2.5e-7 (the fit's largest, its own fp32 roundings included) plus the result's rounding; the left tail to -4
    relative to the value: 4.2e-5 of the fit and 2 P eps = 4e-6 of the exponent's rounding, P = log2 h >= -15.  Zeros stay zeros,
    large values pass or vanish."""
    N = 256
    x = torch.linspace(-9.0, 9.0, M * N, device="cuda:0").reshape(M, N)
    x[0, :8] = torch.tensor([0.0, -0.0, 1e-30, -1e-30, 40.0, -40.0, 3e38, -3e38])
    y = fused_linear_epilogue(x, torch.eye(N, device="cuda:0"), None, [("gelu_erf",)])
    v = x.double()
    ref = v * 0.5 * torch.special.erfc(-v * 0.5 ** 0.5)
    err = (y.double() - ref).abs()
    assert torch.isfinite(y).all()
    assert bool((err <= 2.5e-7 + EPS * ref.abs()).all()), float((err - EPS * ref.abs()).max())
    tail = (v > -4.0) & (v < -1e-3)
    assert bool((err[tail] <= 5e-5 * ref[tail].abs()).all()), float((err[tail] / ref[tail].abs()).max())
    small = v.abs() < 1e-3   # v / 2 to a few roundings: h(0) is exact
    assert bool((err[small] <= 4 * EPS * ref[small].abs()).all())
