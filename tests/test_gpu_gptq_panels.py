"""GPTQ with a panel's sums formed while the panel before it is quantized: one panel (nothing to form), two (nothing
there when the forming begins), three, and so many that the parts between two barriers are uneven and several chunks long.
Every workgroup width adds in the same order, so a narrow weight's result is a slice of a wide one's, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2307_09782_amd import zqfp
from _util import bf16_tensor
from test_gpu_gptq import _hessian, _unpacked, _w

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [128, 256, 384, 640, 1152])
@pytest.mark.parametrize("G,mode", [(32, 1), (64, 2), (128, 1), (256, 2)])
def test_panels(K, G, mode):
    if K % G:
        pytest.skip("K is not a multiple of G")
    N = 40
    W = _w(K, 12400, 7 * K + G)
    U = _hessian(K, K + 1)[2]
    Ud = torch.from_numpy(U.astype(np.float32)).cuda()
    narrow = _unpacked(zqfp.gptq_pack_weight_fp4(bf16_tensor(np.ascontiguousarray(W[:, :N])), Ud, G, mode), K, N, G)
    codes_o, exps_o, c_o, _ = oracle.gptq_fp4(np.ascontiguousarray(W[:, :N]), U, G, mode)
    assert np.array_equal(narrow[2], c_o) and np.array_equal(narrow[0][0], codes_o[0]) and np.array_equal(narrow[1][0], exps_o[0])
    assert np.mean(narrow[0] == codes_o) >= 0.995 and np.mean(narrow[1] == exps_o) >= 0.995
    for wide in (4110, 8300, 12391):
        got = _unpacked(zqfp.gptq_pack_weight_fp4(bf16_tensor(np.ascontiguousarray(W[:, :wide])), Ud, G, mode), K, wide, G)
        for a, b in zip(got, narrow):
            assert np.array_equal(a[..., :N], b)
