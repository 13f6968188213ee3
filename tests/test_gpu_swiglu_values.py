"""The gated unit's binary32 evaluation, its ranges and its binary64 one: every bfloat16 gate value with ordinary, tiny, huge, zero and
infinite second operands, in both kernels (a workgroup per token, a wave per token), against float64 on the CPU."""
import pytest
import torch

from paper_2307_09782_amd import zqfp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ups", [1, 70])
def test_every_gate_value(ups):
    gates = torch.arange(65536, dtype=torch.int32).to(torch.int16).view(torch.bfloat16)
    gen = torch.Generator().manual_seed(ups)
    up = torch.randn(ups * 65536, generator=gen).bfloat16()
    if ups > 1:  # the ends of the range 2^-30 .. 2^30 and what is past them
        special = [0.0, -0.0, 2.0 ** -30, 2.0 ** -31, -(2.0 ** 30), 2.0 ** 31, 1e-39, 3e38, float("inf"), float("nan")]
        up.view(ups, -1)[:len(special)] = torch.tensor(special).bfloat16()[:, None]
    G, Up = gates.repeat(ups).view(16 * ups, 4096), up.view(16 * ups, 4096)
    H = torch.empty(16 * ups, 4096, dtype=torch.bfloat16, device="cuda")
    zqfp.swiglu_quantize_act_fp8(G.cuda(), Up.cuda(), None, H)
    g, u = G.double(), Up.double()
    want = (g / (1.0 + torch.exp(-g)) * u).float().bfloat16()
    got = H.cpu()
    assert torch.equal(got.isnan(), want.isnan())
    ok = ~want.isnan()
    assert torch.equal(got.view(torch.int16)[ok], want.view(torch.int16)[ok])
