"""The packers' 64-column workgroups and units of whole groups and k-tiles, against the oracle, bit for bit: column
counts around a workgroup's edge, and every form of a unit (one k-tile, two, more; one, two or four groups in it)."""
import numpy as np
import pytest
import torch

import oracle
from _util import bf16_tensor, bits_equal_f32
from paper_2307_09782_amd import inputs, zqfp

pytestmark = pytest.mark.gpu


def _weights(K, N, G, seed):
    w = inputs.bf16_bits_to_f32(inputs.make_w(inputs.Config("w", K, N, (1,), G, 1, 0.0, 4, 20.0, seed=seed))).copy()
    w[:G, N // 2] = 0.0              # a zero group
    w[:, N - 1] *= 2.0 ** -120       # a vanishing column: exponents at their clamp, subnormal weights
    if N > 2:
        w[:, 1] = 0.0                # a zero column
        w[-1, 0] = 2.0 ** 100        # one large weight
    return inputs.f32_to_bf16_bits(w)


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("K,N,G", [(128, 1, 128), (128, 63, 64), (256, 64, 32), (256, 65, 128), (512, 129, 256), (768, 80, 384),
                                   (1024, 48, 1024), (1920, 130, 320), (1152, 66, 96), (4096, 191, 128), (384, 66, 384), (2048, 17, 2048),
                                   (896, 64, 896)])
def test_fp4_units_bit_exact(K, N, G, mode):
    W = _weights(K, N, G, K + N)
    packed = zqfp.pack_weight_fp4(bf16_tensor(W), G, mode)
    codes, exps, c = (t.cpu().numpy() for t in zqfp.unpack_codes(packed, K, N, G))
    codes_o, exps_o, c_o, _ = oracle.pack_weight(W, G, mode)
    assert np.array_equal(codes, codes_o) and np.array_equal(exps, exps_o) and bits_equal_f32(c, c_o)
    zqfp.packed_weight_check(packed, K, N, G)
    strips = (N + 15) // 16
    last = packed[256:256 + strips * 8 * K].view(strips, K // 128, 4, 16, 16)[-1, :, :, N - 16 * (strips - 1):]
    assert int(last.count_nonzero()) == 0  # padding columns hold zero codes


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("K,N,G", [(128, 63, 128), (512, 65, 256), (1536, 130, 384), (2048, 64, 128), (384, 20, 384), (1024, 130, 1024),
                                   (2176, 65, 2176)])
def test_fp8_units_bit_exact_rows_of_any_stride(K, N, G, mode):
    W = _weights(K, N, G, K + N)
    wide = torch.zeros((K, N + 3), dtype=torch.bfloat16, device="cuda")  # rows start at any 2-byte address
    wide[:, 1:N + 1] = bf16_tensor(W)
    packed = zqfp.pack_weight_fp8(wide[:, 1:N + 1], G, mode)
    codes, exps, c = (t.cpu().numpy() for t in zqfp.unpack_codes_fp8(packed, K, N, G))
    codes_o, exps_o, c_o, _, _ = oracle.pack_weight_fp8(W, G, mode)
    assert np.array_equal(codes, codes_o) and np.array_equal(exps, exps_o) and bits_equal_f32(c, c_o)
