"""Sorting again after one binning gives the same lists: the sort's input, or
the instances it leaves there, stay in place whatever the number of passes
(tile counts and orders with one, two, three, five and six)."""
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


@pytest.mark.parametrize("sizes,bin_order,persistent,primitive", [
    ([(90, 70)], 0, 0, 0), ([(90, 70), (33, 40)], 1, 1, 0), ([(600, 400)], 0, 0, 0), ([(4112, 4096)], 0, 1, 0),
    ([(90, 70)], 2, 0, 0), ([(90, 70)], 2, 1, 1), ([(600, 400)], 2, 0, 0)])
def test_sort_twice(sizes, bin_order, persistent, primitive):
    scene = S.custom_scene(400, 8, seed=1411, scale_lo=0.02, scale_hi=0.2, primitive=primitive)
    cams = S.make_cameras(sizes, seed=1412)
    rast = snp.Rasterizer(config_for(scene, bin_order=bin_order, persistent=persistent, fwd_cache=0), 400, cams)
    params = snp.params_to_device(scene)
    inst = rast.prepare(params)
    images, T = rast.new_images()
    rast.forward(params, images, T)
    first = [x.clone() for x in (rast.keys(inst), rast.values(inst), rast.ranges(), images, T)]
    for _ in range(2):
        rast.sort()
        images.fill_(-1.0)
        rast.forward(params, images, T)
        for a, b in zip((rast.keys(inst), rast.values(inst), rast.ranges(), images, T), first):
            assert torch.equal(a, b)
