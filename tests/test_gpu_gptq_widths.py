"""GPTQ at every width of a workgroup (16, 32, 48 and 64 output channels, chosen by the channel count): the plain
packer's result under an identity Hessian, bit for bit, and with feedback the oracle's within the bars of
test_gpu_gptq.py."""
import numpy as np
import pytest
import torch

import oracle
from paper_2307_09782_amd import zqfp
from _util import bf16_tensor
from test_gpu_gptq import _hessian, _unpacked, _w

pytestmark = pytest.mark.gpu

# the last workgroup partly filled in each; 256 compute units
SHAPES = [(384, 15), (256, 4110), (512, 4083), (256, 8300), (256, 12391), (256, 16500)]


@pytest.mark.parametrize("K,N", SHAPES)
@pytest.mark.parametrize("G,mode", [(32, 2), (64, 1), (128, 2), (256, 2)])
def test_identity_hessian(K, N, G, mode):
    if K % G:
        pytest.skip("K is not a multiple of G")
    W = _w(K, N, K + N)
    W[W == 0x8000] = 0  # a negative zero loses its sign when zero times an error is added to it
    Wd = bf16_tensor(W)
    got = zqfp.gptq_pack_weight_fp4(Wd, torch.eye(K, dtype=torch.float32, device="cuda"), G, mode)
    for a, b in zip(_unpacked(got, K, N, G), _unpacked(zqfp.pack_weight_fp4(Wd, G, mode), K, N, G)):
        assert np.array_equal(a, b)
    zqfp.packed_weight_check(got, K, N, G)


@pytest.mark.parametrize("K,N,G,mode", [(384, 15, 64, 1), (256, 4110, 32, 1), (256, 8300, 128, 2), (256, 12391, 256, 1), (256, 16500, 64, 2),
                                        (512, 4083, 256, 2)])
def test_feedback(K, N, G, mode):
    W = _w(K, N, 3 * K + N)
    _, _, U = _hessian(K, K)
    codes, exps, c = _unpacked(zqfp.gptq_pack_weight_fp4(bf16_tensor(W), torch.from_numpy(U.astype(np.float32)).cuda(), G, mode), K, N, G)
    codes_o, exps_o, c_o, _ = oracle.gptq_fp4(W, U, G, mode)
    assert np.array_equal(c, c_o) and np.array_equal(codes[0], codes_o[0]) and np.array_equal(exps[0], exps_o[0])
    assert np.mean(codes == codes_o) >= 0.995 and np.mean(exps == exps_o) >= 0.995


@pytest.mark.parametrize("power", [-125, -60, 60, 126])
@pytest.mark.parametrize("mode", [1, 2])
def test_a_power_of_two_on_the_factor_changes_nothing(power, mode):
    """err = (w - q) / U[k][k] and w -= U[k][j] err: a factor 2^n on U cancels exactly, up to the ends of binary32 (at 2^-125
    the reciprocals of diagonals of 1 / 8 are out of range).  U has 8-bit entries of at least 2^-16, so none loses a bit."""
    K, N, G = 256, 100, 64
    Wd = bf16_tensor(_w(K, N, 5))
    U = torch.from_numpy((_hessian(K, K)[2] * 0.125).astype(np.float32)).cuda().bfloat16().float()
    U = torch.where(U.abs() < 2.0 ** -16, torch.zeros_like(U), U).contiguous()
    assert 2.0 ** -20 < U.diagonal().min().item() and U.diagonal().min().item() < 0.5 and U.diagonal().max().item() < 4
    want = zqfp.gptq_pack_weight_fp4(Wd, U, G, mode)
    got = zqfp.gptq_pack_weight_fp4(Wd, (U.double() * 2.0 ** power).float(), G, mode)
    for a, b in zip(_unpacked(got, K, N, G), _unpacked(want, K, N, G)):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("K,N,G", [(256, 100, 64), (512, 4110, 256)])
def test_operands_at_natural_alignment(K, N, G):
    """The factor starts one float into a buffer, the weight one element into each of its rows: the aligned call's blob."""
    W, U = _w(K, N, 9), _hessian(K, K)[2].astype(np.float32)
    wide = torch.zeros((K, N + 3), dtype=torch.bfloat16, device="cuda")
    wide[:, 1:N + 1] = bf16_tensor(W)
    flat = torch.empty(K * K + 1, dtype=torch.float32, device="cuda")
    off = flat[1:].view(K, K)
    off.copy_(torch.from_numpy(U))
    assert off.data_ptr() % 16 == 4
    want = zqfp.gptq_pack_weight_fp4(bf16_tensor(W), torch.from_numpy(U).cuda(), G, 1)
    got = zqfp.gptq_pack_weight_fp4(wide[:, 1:N + 1], off, G, 1)
    for a, b in zip(_unpacked(got, K, N, G), _unpacked(want, K, N, G)):
        assert np.array_equal(a, b)
