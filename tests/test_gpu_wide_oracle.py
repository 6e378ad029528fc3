"""The forward of few tiles against the FP64 oracle: rendered without counting
pairs (a counting forward takes the plain kernel), its images, and its pair
cache through the backward's gradients.  Up to 1.5 tiles per CU: forward of
eight waves per 8 x 8 block, backward a workgroup of eight waves per block; up
to 2: backward of sixteen waves per tile; up to 6: forward of four waves,
backward of eight waves per tile."""
import math

import numpy as np
import pytest
import torch

import synthetic as S
from oracle.render import render_view
from tests.gpu_helpers import IMG_TOL, config_for, grad_parity, options_for, run_forward, say

pytestmark = pytest.mark.gpu

KEYS = ["centers", "scales", "quats", "w1", "b1", "w2", "b2", "colors"]


@pytest.fixture(autouse=True)
def _announce(request):
    say(f"[gpu-test] {request.node.name}")
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("N,fwd_cache,tiles_per_cu,dense", [
    (4, 1, 0, False), (16, 1, 0, True), (32, 0, 0, True), (4, 1, 2, True), (16, 0, 2, False), (32, 1, 2, False),
    (32, 0, 2, True), (4, 0, 4, False), (8, 1, 4, True)])
def test_uncounted_forward(N, fwd_cache, tiles_per_cu, dense):
    lo, hi = (0.1, 0.35) if dense else (0.02, 0.15)
    scene = S.custom_scene(120, N, seed=2201 + N, scale_lo=lo, scale_hi=hi)
    sizes = [(73, 57), (18, 41)]
    if tiles_per_cu:  # one view of that many tiles, its last column and row a pixel wide
        cus = torch.cuda.get_device_properties(0).multi_processor_count
        side = int(math.sqrt(tiles_per_cu * cus)) - 1
        sizes = [(16 * side + 1, 16 * side + 1)]
        assert (side + 1) ** 2 > (1.5 if tiles_per_cu == 2 else 2.5) * cus
    cams = S.make_cameras(sizes, seed=2202)
    cfg = config_for(scene, tile=(16, 16, 1), fwd_cache=fwd_cache)
    fw = run_forward(scene, cams, cfg, count_pairs=False)
    for v, cam in enumerate(cams):
        ref = render_view(scene, cam, options_for(cfg))
        err, terr = np.max(np.abs(fw["images"][v] - ref["image"])), np.max(np.abs(fw["T"][v] - ref["T"]))
        say(f"  view {v}: image err {err:.2e}, T err {terr:.2e}")
        assert err <= IMG_TOL and terr <= IMG_TOL
    grad_parity(scene, cams, S.make_targets(cams, seed=2203), cfg, KEYS, fw=fw)
