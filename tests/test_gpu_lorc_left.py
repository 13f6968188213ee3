"""The left factor T = y . U in the ways it is formed (a workgroup per 4 or 8 ranks, all sums in one
workgroup, a launch of its own) and behind every producer; codes, scales and H must be those of the call without a factor, bit for bit.
y is the bfloat16 value that the quantizer sees, taken from the library where it returns it and formed in torch otherwise; T against
float64: products are exact in binary64, so |err| <= 2^-18 * sum|y u| leaves room for the order of the binary32 additions."""
import pytest
import torch

from paper_2307_09782_amd import zqfp

pytestmark = pytest.mark.gpu


def _inputs(M, K, r, ldx=0):
    gen = torch.Generator(device="cuda").manual_seed(M + 3 * K + r)
    X = torch.randn(M, K + ldx, generator=gen, device="cuda").bfloat16()[:, :K]
    O = torch.randn(M, K + ldx, generator=gen, device="cuda").bfloat16()[:, :K]
    gain = (1 + 0.1 * torch.randn(K, generator=gen, device="cuda")).bfloat16()
    bias = (0.1 * torch.randn(K, generator=gen, device="cuda")).bfloat16()
    U = (torch.randn(K, r, generator=gen, device="cuda") * 0.01).half()
    return X, O, gain, bias, U


def _check(T, y, U):
    ref, mag = y.double() @ U.double(), y.double().abs() @ U.double().abs()
    worst = ((T.double() - ref).abs() / mag.clamp_min(1e-300)).max().item()
    assert worst <= 2.0 ** -18, worst


# tokens around the lines between the forms (16 per workgroup apart), ranks that end inside a block of 8 or 16
@pytest.mark.parametrize("K", [128, 1408, 8320])
@pytest.mark.parametrize("M,r", [(2, 4), (40, 8), (70, 4), (20, 12), (1, 9), (3, 16), (64, 16), (65, 16), (17, 40), (33, 64), (50, 23), (129, 40), (300, 33), (513, 12), (600, 16), (820, 10), (801, 17), (830, 64), (2050, 48)])
def test_plain_and_relu(M, K, r):
    X, _, _, _, U = _inputs(M, K, r, ldx=64)
    y = X.clamp_min(0)
    Xq, sx, T = zqfp.relu_quantize_act_fp8(X, U)
    for a, b in zip((Xq, sx), zqfp.relu_quantize_act_fp8(X)):
        assert torch.equal(a, b)
    _check(T, y, U)
    X = X.contiguous()
    Xq, sx, T = zqfp.quantize_act_fp8(X, U)
    for a, b in zip((Xq, sx), zqfp.quantize_act_fp8(X)):
        assert torch.equal(a, b)
    _check(T, X, U)


@pytest.mark.parametrize("K", [384, 4096, 8448])
@pytest.mark.parametrize("M,r", [(16, 8), (2, 16), (5, 40), (64, 64), (300, 40), (400, 64), (530, 16), (1100, 24), (1450, 9)])
def test_producers(M, K, r):
    X, O, gain, bias, U = _inputs(M, K, r)
    # a row whose residual is its negative is zero: the normalisation of zeros (RMS) and the bias alone (layer norm)
    O[M // 2] = -X[M // 2]
    H, Xq, sx, T = zqfp.add_norm_quantize_act_fp8(X, O, gain, 1e-5, None, U)
    for a, b in zip((H, Xq, sx), zqfp.add_norm_quantize_act_fp8(X, O, gain, 1e-5)):
        assert torch.equal(a, b)
    hd = H.double()
    rstd = 1 / torch.sqrt(hd.square().mean(1, keepdim=True).float() + 1e-5)
    _check(T, ((H.float() * rstd) * gain.float()).bfloat16(), U)
    Hl, Xl, sl, Tl = zqfp.add_norm_quantize_act_fp8(X, O, gain, 1e-5, bias, U)
    for a, b in zip((Hl, Xl, sl), zqfp.add_norm_quantize_act_fp8(X, O, gain, 1e-5, bias)):
        assert torch.equal(a, b)
    mean = hd.mean(1, keepdim=True)
    var = (hd.square().mean(1, keepdim=True) - mean * mean).clamp_min(0)
    rstd = 1 / torch.sqrt(var.float() + 1e-5)
    _check(Tl, (((H.float() - mean.float()) * rstd) * gain.float() + bias.float()).bfloat16(), U)
    # without a residual: the same as with H for X
    for a, b in zip((Xq, sx, T), zqfp.rmsnorm_quantize_act_fp8(H, gain, 1e-5, U)):
        assert torch.equal(a, b)
    for a, b in zip((Xl, sl, Tl), zqfp.layernorm_quantize_act_fp8(H, gain, bias, 1e-5, U)):
        assert torch.equal(a, b)
    # in place, over the residual stream and over the gate: codes, scales and H as before, T within tolerance of the same y
    R = O.clone()
    out = zqfp.add_norm_quantize_act_fp8(X, R, gain, 1e-5, None, U, H=R)
    for a, b in zip(out[:3], (H, Xq, sx)):
        assert torch.equal(a, b)
    _check(out[3], ((H.float() * (1 / torch.sqrt(hd.square().mean(1, keepdim=True).float() + 1e-5))) * gain.float()).bfloat16(), U)
    P = torch.empty_like(X)
    Xs, ss, Ts = zqfp.swiglu_quantize_act_fp8(X, O, U, H=P)
    _check(Ts, P, U)
    for a, b in zip((Xs, ss), zqfp.swiglu_quantize_act_fp8(X, O)):
        assert torch.equal(a, b)
    _check(zqfp.swiglu_quantize_act_fp8(X, O, U)[2], P, U)
    gate = X.clone()
    out = zqfp.swiglu_quantize_act_fp8(gate, O, U, H=gate)
    assert torch.equal(gate, P) and torch.equal(out[0], Xs) and torch.equal(out[1], ss)
    _check(out[2], P, U)


def test_an_infinite_entry_of_u_gives_infinities():
    for M in (4, 700, 900):
        X, _, _, _, U = _inputs(M, 1152, 20)
        X = X.abs().contiguous() + 1
        U[300, 18] = float("inf")
        T = zqfp.quantize_act_fp8(X, U)[2]
        assert bool((T[:, 18] == float("inf")).all()) and bool(torch.isfinite(T[:, :18]).all()) and bool(torch.isfinite(T[:, 19]).all())
