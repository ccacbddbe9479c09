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


@pytest.mark.parametrize("M", [8, 128, 2048])
def test_gelu_erf_far_left_tail_keeps_its_relative_accuracy(M):
    """Behind -6 the values are tiny and an absolute bound says nothing.  Each bound is the fit's error there plus a few roundings of
    the exponent (up to 120, so 120 x 2^-24 each, 1e-5 of the value); at -12.5 the last normal numbers are near."""
    N = 256
    x = -torch.linspace(0.5, 12.5, M * N, device="cuda:0").reshape(M, N)
    y = fused_linear_epilogue(x, torch.eye(N, device="cuda:0"), None, [("gelu_erf",)])
    v = x.double()
    ref = v * 0.5 * torch.special.erfc(-v * 0.5 ** 0.5)
    rel = ((y.double() - ref) / ref).abs()
    for upto, bound in ((4.0, 5e-5), (6.0, 2e-3), (8.0, 2.3e-3), (12.5, 8e-3)):
        assert bool((rel[v >= -upto] <= bound).all()), (upto, float(rel[v >= -upto].max()))


@pytest.mark.parametrize("M", [8, 128, 2048])
def test_gelu_erf_of_a_value_does_not_depend_on_its_neighbours(M):
    """Values behind 6 take another form, which the tiled kernels run only where there are any: near values come out the same bits."""
    N = 256
    x = torch.linspace(-5.9, 5.9, M * N, device="cuda:0").reshape(M, N)
    far = x.clone()
    far[::7, ::5] = -7.0
    near = fused_linear_epilogue(x, torch.eye(N, device="cuda:0"), None, [("gelu_erf",)])
    mixed = fused_linear_epilogue(far, torch.eye(N, device="cuda:0"), None, [("gelu_erf",)])
    same = far == x
    assert torch.equal(near[same], mixed[same])
    assert bool((mixed[~same] == mixed[0, 0]).all()) and float(mixed[0, 0]) < 0.0
