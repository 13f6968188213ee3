"""Every kernel behind the GEMM calls on a shape that reaches it: the form the library names is asserted, so that a change
of the dispatch cannot leave a kernel untested.  Tolerances are those of test_gpu_parity.py."""
import numpy as np
import pytest
import torch

from paper_2307_09782_amd import inputs, zqfp
from _util import bf16_tensor, check_gemm
from test_gpu_parity import _check_bf16, _gemm_case, _sync_np, _weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("M,K,N,G,mode,r", [(16, 24704, 4090, 128, 2, 8),   # 193 k-tiles: chunks of 49, 49, 49, 46
                                            (9, 24704, 4096, 128, 1, 0),
                                            (5, 8320, 12304, 64, 2, 8),     # 65 k-tiles: chunks of 33 and 32
                                            (7, 8448, 12292, 128, 1, 16)])  # a rank beyond the registers' eight
def test_decode_form_in_chunks(M, K, N, G, mode, r, out_dtype):
    """At most 16 tokens, K beyond 64 k-tiles in chunks through the workspace, scales and LoRC in the reduce kernel; the
    same call without a workspace is served by another kernel."""
    assert zqfp.probe_gemm_form(M, K, N, G, r=r) == zqfp.FORM_DECODE
    assert zqfp.probe_gemm_form(M, K, N, G, r=r, have_workspace=False) == zqfp.FORM_MID
    assert zqfp.gemm_workspace_bytes(M, K, N) == -(-K // 128 // 64) * M * (-(-N // 16) * 16) * 4
    Y, Y_o, Sabs = _gemm_case(M, K, N, G, mode, r, seed_cfg="llama70b_ffn_decode", full=False, nsamples=2048, out_dtype=out_dtype)
    if out_dtype == torch.float32:
        check_gemm(Y, Y_o, Sabs, f"decode chunks M{M} K{K} N{N}")
    else:
        _check_bf16(Y, Y_o, Sabs, f"decode chunks, bf16, M{M} K{K} N{N}")


@pytest.mark.parametrize("M,K,N,G,mode,r", [(16, 256, 4100, 128, 1, 0), (3, 5120, 96, 128, 2, 5), (4, 8192, 80, 128, 1, 8)])
def test_decode_form_in_one_piece(M, K, N, G, mode, r):
    assert zqfp.probe_gemm_form(M, K, N, G, r=r) == zqfp.FORM_DECODE and zqfp.gemm_workspace_bytes(M, K, N) == 0
    Y, Y_o, Sabs = _gemm_case(M, K, N, G, mode, r)
    check_gemm(Y, Y_o, Sabs, f"decode M{M} K{K} N{N}")


@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("M,K,N,G,mode,r", [(33, 11008, 256, 128, 2, 0),    # a down projection's K (86 k-tiles): uneven slices
                                            (100, 14336, 136, 128, 1, 3),   # ragged tokens and channels
                                            (64, 11008, 512, 128, 1, 8),
                                            (257, 512, 4000, 128, 2, 8)])   # not split: the smallest tiles
def test_tiled_form_with_and_without_k_slices(M, K, N, G, mode, r, out_dtype):
    """The planner's K slices through the workspace, and the same call un-split without one."""
    assert zqfp.probe_gemm_form(M, K, N, G, r=r) == zqfp.FORM_TILE
    split = K > 8192
    assert (zqfp.gemm_workspace_bytes(M, K, N) > 0) == split
    Y, Y_o, Sabs = _gemm_case(M, K, N, G, mode, r, out_dtype=out_dtype)
    what = f"tiles M{M} K{K} N{N} {out_dtype}"
    if out_dtype == torch.bfloat16:
        return _check_bf16(Y, Y_o, Sabs, what)
    check_gemm(Y, Y_o, Sabs, what)
    if split and not r:
        assert zqfp.probe_gemm_form(M, K, N, G, have_workspace=False) == zqfp.FORM_TILE
        cfg = inputs.CONFIGS["tiny"]
        cfg = inputs.Config(cfg.name, K, N, (M,), G, mode, cfg.outlier_frac, cfg.outlier_count, cfg.outlier_gain, r, cfg.seed)
        Xq, sx = zqfp.quantize_act_fp8(bf16_tensor(inputs.make_x(cfg, M)))
        plain = _sync_np(zqfp.w4a8_gemm(Xq, sx, _weights(cfg, G, mode)[1], N, G, workspace=False))
        check_gemm(plain, Y_o, Sabs, what + ", no workspace")


@pytest.mark.parametrize("form,M,K,N,r,accum", [
    (zqfp.FORM_STREAM, 9, 9216, 8192, 0, 0), (zqfp.FORM_STREAM, 24, 1024, 1040, 8, 0), (zqfp.FORM_STREAM, 17, 2048, 4090, 0, 0),
    (zqfp.FORM_STREAM, 32, 4096, 4096, 4, 1), (zqfp.FORM_MID, 32, 4096, 4096, 8, 1), (zqfp.FORM_MID, 12, 9216, 8192, 0, 0),
    (zqfp.FORM_MID, 64, 1024, 16384, 4, 1), (zqfp.FORM_DECODE, 16, 5120, 1040, 40, 0), (zqfp.FORM_TILE, 257, 256, 8200, 8, 0)])
def test_fp8_weights_on_every_form(form, M, K, N, r, accum):
    """E4M3 weights against the plain definition in float64 with the codes that the packer wrote; bound as in test_gpu_w8a8.py."""
    assert zqfp.probe_gemm_form(M, K, N, 128, 8, r, accum) == form
    gen = torch.Generator(device="cuda").manual_seed(M + K + N)
    packed = zqfp.pack_weight_fp8((torch.randn(K, N, generator=gen, device="cuda") * 0.02).bfloat16(), 128, 1)
    Xq, sx = zqfp.quantize_act_fp8(torch.randn(M, K, generator=gen, device="cuda").bfloat16())
    T = torch.randn(M, r, generator=gen, device="cuda") if r else None
    V = (torch.randn(r, N, generator=gen, device="cuda") * 0.1).half() if r else None
    Y = zqfp.w8a8_gemm(Xq, sx, packed, N, 128, T, V, accum=accum).double()
    codes, exps, c = zqfp.unpack_codes_fp8(packed, K, N, 128)
    w = codes.view(torch.float8_e4m3fn).double() * torch.exp2(exps.double() - 127).repeat_interleave(128, 0) * c.double()
    a = Xq.view(torch.float8_e4m3fn).double() * sx.double()[:, None]
    ref, mag = a @ w, a.abs() @ w.abs()
    if r:
        ref, mag = ref + T.double() @ V.double(), mag + T.double().abs() @ V.double().abs()
    assert bool(((Y - ref).abs() <= 7 * 2.0 ** -13 * mag).all())
