"""The low-rank correction in every GEMM epilogue at the ranks where its handling changes: part of a step of four, whole steps,
the second slot of a wave (beyond 32), a second block of ranks in LDS (beyond 32), the largest; shapes that reach each kernel.
Tolerance and reference as in test_gpu_gemm_mid.py: float64 with the codes that the packer wrote, |err| <= 2^-18 * sum|terms|."""
import pytest
import torch

from paper_2307_09782_amd import zqfp
from test_gpu_gemm_mid import _check

pytestmark = pytest.mark.gpu
RANKS = [1, 4, 7, 8, 9, 31, 32, 33, 40, 64]


@pytest.mark.parametrize("r", RANKS)
def test_decode_form(r):
    for M, K, N in ((16, 1024, 520), (5, 3584, 4130), (16, 8192, 8200)):  # the last: eight k-tiles per wave, upper band in LDS
        assert zqfp.probe_gemm_form(M, K, N, r=r) == zqfp.FORM_DECODE
        _check(M, K, N, 128, 1, r, 4)
    _check(3, 1280, 200, 128, 1, r, 8)


@pytest.mark.parametrize("r", [5, 8, 40, 64])
def test_decode_form_with_sixteen_waves(r):
    try:
        zqfp.probe_force_decode_waves(16)
        _check(9, 2048, 1040, 128, 1, r, 4)
    finally:
        zqfp.probe_force_decode_waves(8)


@pytest.mark.parametrize("r", RANKS)
def test_sums_of_chunks_and_slices(r):
    assert zqfp.probe_gemm_form(7, 8448, 12292, r=r) == zqfp.FORM_DECODE and zqfp.gemm_workspace_bytes(7, 8448, 12292) > 0
    _check(7, 8448, 12292, 128, 1, r, 4)                      # channels on 8 bytes
    _check(33, 11008, 262, 128, 2, r, 4, torch.bfloat16)      # and not


@pytest.mark.parametrize("bm,bn,kg", [(64, 128, 1), (64, 128, 2), (64, 192, 2), (64, 256, 1), (128, 128, 1), (128, 192, 1), (128, 256, 1), (256, 256, 1)])
def test_tiled_form(bm, bn, kg):
    try:
        zqfp.probe_force_tile_plan(bm, bn, 1, kg)
        for r in RANKS:
            _check(300, 512, 550, 128, 1, r, 4)
        if bn == 128:
            for r in (8, 33, 64):
                _check(300, 512, 550, 128, 1, r, 8)
    finally:
        zqfp.probe_force_tile_plan()


def test_infinite_factors_stay_in_their_row_and_column():
    """Padding ranks multiply nothing: an infinite entry of V or T gives infinities of the right sign where the definition has
    them and leaves every other output finite."""
    for M, K, N in ((4, 512, 64), (200, 512, 520)):
        gen = torch.Generator(device="cuda").manual_seed(1)
        packed = zqfp.pack_weight_fp4((torch.randn(K, N, generator=gen, device="cuda") * 0.02).bfloat16(), 128, 1)
        Xq, sx = zqfp.quantize_act_fp8(torch.randn(M, K, generator=gen, device="cuda").bfloat16())
        T = torch.rand(M, 5, generator=gen, device="cuda") + 0.5
        V = torch.ones(5, N, device="cuda").half()
        V[4, 3] = float("inf")
        T[2, 0] = -float("inf")
        Y = zqfp.w4a8_gemm_lorc(Xq, sx, packed, N, 128, T, V)
        want = torch.zeros(M, N, device="cuda")
        want[:, 3] = float("inf")
        want[2] = -float("inf")
        want[2, 3] = float("nan")
        assert torch.equal(torch.isnan(Y), torch.isnan(want)) and torch.equal(torch.isinf(Y), torch.isinf(want))
        assert torch.equal(torch.sign(Y)[torch.isinf(want)], torch.sign(want)[torch.isinf(want)])
