"""Launches of up to six tiles per CU, through each of the backward's splits of
a 16 x 16 tile (a workgroup per 8 x 8 block, sixteen or eight waves per tile)
against the FP64 oracle, and the forward's: ragged edges with blocks wholly
outside the image, more instances than a batch, pixels that end early."""
import math

import pytest
import torch

import synthetic as S
from tests.gpu_helpers import check_images, config_for, grad_parity, run_forward, say

pytestmark = pytest.mark.gpu

KEYS = ["centers", "scales", "quats", "w1", "b1", "w2", "b2", "colors"]


@pytest.fixture(autouse=True)
def _announce(request):
    say(f"[gpu-test] {request.node.name}")
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("N,fwd_cache,tiles_per_cu,dense", [
    (4, 1, 0, False), (8, 0, 0, True), (16, 1, 0, True), (32, 1, 0, False), (8, 1, 2, False), (16, 0, 4, False)])
def test_splits_of_a_tile(N, fwd_cache, tiles_per_cu, dense):
    lo, hi = (0.1, 0.35) if dense else (0.02, 0.15)
    scene = S.custom_scene(120, N, seed=1611 + N, scale_lo=lo, scale_hi=hi)
    sizes = [(73, 57), (18, 41)]
    if tiles_per_cu:  # one view of that many tiles, its last column and row a pixel wide
        cus = torch.cuda.get_device_properties(0).multi_processor_count
        side = int(math.sqrt(tiles_per_cu * cus)) - 1
        sizes = [(16 * side + 1, 16 * side + 1)]
    cams = S.make_cameras(sizes, seed=1512)
    targets = S.make_targets(cams, seed=1513)
    cfg = config_for(scene, tile=(16, 16, 1), fwd_cache=fwd_cache)
    fw = run_forward(scene, cams, cfg)
    check_images(fw, scene, cams, cfg)
    grad_parity(scene, cams, targets, cfg, KEYS, fw=fw)
