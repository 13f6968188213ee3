"""RMS normalisation with the rank-8 left factor, rows that end inside a wave's first 512 elements, just behind them and
beyond one chunk per thread, with one token and with enough for the narrow workgroups: codes and scales those of the call
without the factor, T within the rounding of its float32 sums (K additions of relative error 2^-24 each at most)."""
import pytest
import torch

from paper_2307_09782_amd import zqfp

pytestmark = pytest.mark.gpu


def _check_t(T, x, gain, U):
    """T against the normalised row, to bfloat16 as the kernel rounds it"""
    rstd = 1.0 / torch.sqrt((x.double() ** 2).mean(1, keepdim=True).float() + 1e-5)
    y = ((x.float() * rstd) * gain.float()).bfloat16().double()
    ref, mag = y @ U.double(), y.abs() @ U.double().abs()
    # a value of y may round the other way where torch's root or quotient differ in the last bit: one bfloat16 step of it
    assert bool(((T.double() - ref).abs() <= mag * (x.shape[1] * 2.0 ** -24) + (y.abs() * 2.0 ** -8).amax(1, keepdim=True) * U.double().abs().amax()).all())


@pytest.mark.parametrize("K", [128, 640, 1920, 2176, 8320])
@pytest.mark.parametrize("M", [1, 70])
def test_rms_rank8_rows(M, K):
    gen = torch.Generator(device="cuda").manual_seed(K + M)
    X = torch.randn(M, K, generator=gen, device="cuda").bfloat16()
    gain = (1 + 0.1 * torch.randn(K, generator=gen, device="cuda")).bfloat16()
    U = (torch.randn(K, 8, generator=gen, device="cuda") * 0.1).half()
    Xq, sx, T = zqfp.rmsnorm_quantize_act_fp8(X, gain, 1e-5, U)
    Xq0, sx0 = zqfp.rmsnorm_quantize_act_fp8(X, gain, 1e-5)
    assert torch.equal(Xq, Xq0) and torch.equal(sx, sx0)
    _check_t(T, X, gain, U)


# both sides of the rules that load U ahead in 1024 threads: row lengths around 4096, 8192, 12288 and 16384, tokens around 256
@pytest.mark.parametrize("K", [4096, 4224, 8320, 12416, 16512])
@pytest.mark.parametrize("M", [3, 257])
def test_residual_rms_rank8_rows(M, K):
    gen = torch.Generator(device="cuda").manual_seed(K + M)
    X, R = (torch.randn(M, K, generator=gen, device="cuda").bfloat16() for _ in range(2))
    gain = (1 + 0.1 * torch.randn(K, generator=gen, device="cuda")).bfloat16()
    U = (torch.randn(K, 8, generator=gen, device="cuda") * 0.1).half()
    H, Xq, sx, T = zqfp.add_norm_quantize_act_fp8(X, R, gain, 1e-5, None, U)
    H0, Xq0, sx0 = zqfp.add_norm_quantize_act_fp8(X, R, gain, 1e-5, None, None)
    assert torch.equal(H, H0) and torch.equal(Xq, Xq0) and torch.equal(sx, sx0)
    Xq1, sx1, T1 = zqfp.rmsnorm_quantize_act_fp8(H, gain, 1e-5, U)
    assert torch.equal(Xq, Xq1) and torch.equal(sx, sx1)
    _check_t(T, H, gain, U)
    _check_t(T1, H, gain, U)
