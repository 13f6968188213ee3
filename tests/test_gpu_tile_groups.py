"""Wave groups of the tiled kernel that take the k-tiles in turn: every remainder of k-tiles over two and four groups (the first
groups then multiply zeros in their first step), pipelines shorter than the LDS stages, K slices that start inside a group of
scales, all group kinds (several per k-tile, one, one over several k-tiles), ragged tokens and channels, ranks of the correction that the
groups share out.  Reference and tolerance as in test_gpu_gemm_mid.py."""
import pytest
import torch

from paper_2307_09782_amd import zqfp
from test_gpu_gemm_mid import _check

pytestmark = pytest.mark.gpu


@pytest.fixture(params=[(64, 64, 4), (64, 96, 4), (64, 128, 4), (64, 128, 2), (64, 192, 2), (64, 256, 2)], ids=lambda p: "x".join(map(str, p)))
def shape(request):
    yield request.param
    zqfp.probe_force_tile_plan()


@pytest.mark.parametrize("nkt", [1, 2, 3, 4, 5, 6, 7, 11, 13, 16])
def test_every_remainder_of_k_tiles(shape, nkt):
    bm, bn, kg = shape
    zqfp.probe_force_tile_plan(bm, bn, 1, kg)
    _check(150, 128 * nkt, 296, 128, 1, 0, 4)
    _check(65, 128 * nkt, 130, 32, 2, 9, 4, torch.bfloat16)
    _check(70, 128 * nkt, 200, 128 * nkt, 1, 8, 4, accum=zqfp.ACCUM_FAST)
    if (bn, kg) == (128, 2):
        _check(150, 128 * nkt, 296, 128, 1, 3, 8)
        _check(70, 128 * nkt, 200, 128 * nkt, 2, 0, 8, accum=zqfp.ACCUM_FAST)


@pytest.mark.parametrize("G", [64, 384])
@pytest.mark.parametrize("ksplit", [2, 3, 5])
def test_slices_that_do_not_come_out_even(shape, ksplit, G):
    bm, bn, kg = shape
    zqfp.probe_force_tile_plan(bm, bn, ksplit, kg)
    assert zqfp.gemm_workspace_bytes(90, 2688, 210) == -(-21 // -(-21 // ksplit)) * 90 * 224 * 4
    _check(90, 2688, 210, G, 1, 4, 4)


def test_planner_takes_them():
    """Where they win, and the estimate says so: a few tiles on a short and on a long K."""
    for M, K, N, kg in ((150, 4096, 4096, 4), (257, 11008, 4096, 4), (100, 4096, 12288, 4)):
        assert zqfp.probe_gemm_form(M, K, N) == zqfp.FORM_TILE
        assert zqfp.probe_tile_plan(M, K, N)[2] == kg
        _check(M, K, N, 128, 1, 0, 4)
