"""Gaussian frames where a wave is one 8 x 8 block take an instance's pixels
from a mask: against the tile shape whose lanes test the rectangle themselves,
bit for bit, images and counted pairs -- footprints from one pixel to the whole
view, up to several batches of 256 instances per tile, ragged edges, and
scenes that end within a group of 64 instances or not at all."""
import pytest
import torch

import paper_2510_08491_amd as snp
import synthetic as S
from tests.gpu_helpers import config_for, say

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _announce(request):
    say(f"[gpu-test] {request.node.name}")
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("P,lo,hi,tile,persistent,options", [
    (1, 0.3, 0.4, (16, 16, 1), 0, {}), (64, 0.002, 0.01, (16, 16, 1), 1, {"alpha_min": 1.0 / 255.0}),
    (700, 0.1, 0.6, (16, 16, 1), 0, {"t_eps": 0.0}), (2000, 0.02, 0.3, (16, 16, 1), 1, {}),
    (900, 0.05, 0.4, (8, 8, 1), 0, {"alpha_max": 0.6}), (3000, 0.004, 0.1, (8, 8, 1), 1, {"alpha_min": 0.05})])
def test_masks_match_the_rectangle_tests(P, lo, hi, tile, persistent, options):
    scene = S.custom_scene(P, 8, seed=1211 + P, scale_lo=lo, scale_hi=hi, primitive=1)
    cams = S.make_cameras([(93, 61), (17, 70), (5, 3)], seed=1212)
    params = snp.params_to_device(scene)
    got = []
    for shape in (tile, (16, 16, 2)):
        rast = snp.Rasterizer(config_for(scene, tile=shape, persistent=persistent, **options), P, cams)
        rast.prepare(params)
        images, T = rast.new_images()
        rast.forward(params, images, T)
        counted, T2 = rast.new_images()
        rast.forward(params, counted, T2, count_pairs=True)
        assert torch.equal(images, counted) and torch.equal(T, T2)
        c = rast.counters()
        got.append((images, T, c["hit_pairs"], c["live_pairs"]))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    assert got[0][2:] == got[1][2:]
