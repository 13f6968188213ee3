"""The GEMM form for a few dozen tokens: every block count of 16 tokens, every strip count per workgroup, tokens and
channels that end inside a block, K of fewer k-tiles than waves and of odd numbers of them, all group kinds (several
groups per k-tile, a group count that is no power of two), low-rank corrections held and looped over, both weight
formats, against the plain definition in float64 with the codes that the packer wrote.

FP4 weights: products are exact, so only the float32 additions round: |err| <= 2^-18 * sum|a w| like every exact form.
FP8 weights lose up to 7 * 2^-13 of a run's largest product.  bfloat16 output adds half an ulp."""
import pytest
import torch

from paper_2307_09782_amd import zqfp

pytestmark = pytest.mark.gpu


def _check(M, K, N, G, mode, r, wbits, out_dtype=torch.float32, accum=zqfp.ACCUM_EXACT):
    gen = torch.Generator(device="cuda").manual_seed(M + 7 * K + 13 * N + r)
    W = (torch.randn(K, N, generator=gen, device="cuda") * 0.02).bfloat16()
    X = (torch.randn(M, K, generator=gen, device="cuda") * torch.exp(torch.randn(M, 1, generator=gen, device="cuda"))).bfloat16()
    T = torch.randn(M, r, generator=gen, device="cuda") if r else None
    V = (torch.randn(r, N, generator=gen, device="cuda") * 0.1).half() if r else None
    Xq, sx = zqfp.quantize_act_fp8(X)
    if wbits == 8:
        packed = zqfp.pack_weight_fp8(W, G, mode)
        codes, exps, c = zqfp.unpack_codes_fp8(packed, K, N, G)
        q = codes.view(torch.float8_e4m3fn).double()
        Y = zqfp.w8a8_gemm(Xq, sx, packed, N, G, T, V, out_dtype=out_dtype, accum=accum)
    else:
        packed = zqfp.pack_weight_fp4(W, G, mode)
        codes, exps, c = zqfp.unpack_codes(packed, K, N, G)
        grid = torch.tensor([0, 0.5, 1, 1.5, 2, 3, 4, 6], device="cuda", dtype=torch.float64)
        q = torch.cat([grid, -grid])[codes.long()]
        Y = zqfp.w4a8_gemm_lorc(Xq, sx, packed, N, G, T, V, out_dtype=out_dtype, accum=accum) if r else \
            zqfp.w4a8_gemm(Xq, sx, packed, N, G, out_dtype=out_dtype, accum=accum)
    w = q * torch.exp2(exps.double() - 127).repeat_interleave(G, 0) * c.double()
    a = Xq.view(torch.float8_e4m3fn).double() * sx.double()[:, None]
    ref, mag = a @ w, a.abs() @ w.abs()
    if r:
        ref, mag = ref + T.double() @ V.double(), mag + T.double().abs() @ V.double().abs()
    exact = accum == zqfp.ACCUM_EXACT and wbits == 4
    bound = mag * (2.0 ** -18 if exact else 7 * 2.0 ** -13)
    if out_dtype == torch.bfloat16:
        bound = bound + (ref.abs() + bound) * 2.0 ** -8
    err = (Y.double() - ref).abs()
    assert bool((err <= bound).all()), f"worst err/bound {(err / bound.clamp_min(1e-300)).max().item():.3g}"


# N picks the strips per workgroup: 4096 channels are one round of compute units with one strip, 8192 with two, ...
@pytest.mark.parametrize("wbits", [4, 8])
@pytest.mark.parametrize("N", [16, 50, 1000, 4112, 8200, 12288, 16380])
@pytest.mark.parametrize("M", [17, 33, 64, 65])
def test_token_blocks_and_strips(M, N, wbits):
    _check(M, 2048 if wbits == 8 and M <= 32 else 384, N, 128, 1, 8, wbits)


@pytest.mark.parametrize("wbits", [4, 8])
@pytest.mark.parametrize("M,K,N,G,mode,r", [(20, 128, 272, 128, 1, 0), (40, 1024, 130, 128, 2, 3),
                                            (64, 1152, 1000, 384, 2, 40), (48, 3456, 520, 128, 1, 16), (130, 2176, 300, 128, 1, 0),
                                            (200, 1280, 1024, 256, 2, 8), (16, 8320, 200, 128, 1, 8), (1, 8448, 4100, 256, 1, 0),
                                            (13, 5120, 1040, 128, 2, 40), (4, 8832, 8208, 128, 1, 0), (700, 512, 1024, 128, 1, 0)])
def test_ragged_k_groups_and_ranks(M, K, N, G, mode, r, wbits):
    _check(M, K, N, G, mode, r, wbits)
    _check(M, K, N, G, mode, r, wbits, torch.bfloat16, zqfp.ACCUM_FAST)


# fewer than 64 channels: 16 to 64 tokens per workgroup, whichever starts the most at once, ragged at both ends
@pytest.mark.parametrize("wbits", [4, 8])
@pytest.mark.parametrize("M,K,N,r", [(300, 512, 16, 0), (257, 512, 48, 8), (4100, 640, 48, 0), (1023, 2176, 33, 3), (5000, 384, 63, 0)])
def test_many_tokens_on_a_few_channels(M, K, N, r, wbits):
    assert zqfp.probe_gemm_form(M, K, N, 128, wbits, r) == zqfp.FORM_MID
    _check(M, K, N, 128, 1, r, wbits)


@pytest.mark.parametrize("G", [32, 64])
def test_several_groups_per_k_tile(G):
    _check(50, 1408, 600, G, 1, 0, 4)


def test_a_wider_row_stride_of_the_output_is_left_alone():
    gen = torch.Generator(device="cuda").manual_seed(3)
    M, K, N = 37, 640, 100
    packed = zqfp.pack_weight_fp4((torch.randn(K, N, generator=gen, device="cuda") * 0.02).bfloat16(), 128, 1)
    Xq, sx = zqfp.quantize_act_fp8(torch.randn(M, K, generator=gen, device="cuda").bfloat16())
    Y = zqfp.w4a8_gemm(Xq, sx, packed, N, 128)
    wide = torch.full((M + 2, 160), 7.0, device="cuda")
    zqfp.w4a8_gemm(Xq, sx, packed, N, 128, out=wide[:M, :N])
    assert torch.equal(wide[:M, :N], Y) and bool((wide[:, N:] == 7.0).all()) and bool((wide[M:] == 7.0).all())
