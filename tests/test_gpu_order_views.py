"""Pairs ordered by one workgroup per view: several views, sizes around a
workgroup's keys, depths from one value to many octaves (one to four passes
over the differences to the least), views that see nothing."""
import numpy as np
import pytest
import torch

import paper_2510_08491_amd as snp
import synthetic as S
from tests.gpu_helpers import config_for, say
from tests.test_gpu_order import expected

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _announce(request):
    say(f"[gpu-test] {request.node.name}")
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("P,views,spread", [
    (1, 3, 1.0), (64, 2, 0.0), (1024, 5, 1e-5), (1025, 3, 1e-3), (7919, 2, 1.0), (16384, 2, 30.0), (16385, 2, 1.0),
    (16384, 9, 1.0), (300, 40, 1.0), (5, 1, 0.0)])
def test_views_ordered_apart_match_a_host_sort(P, views, spread):
    scene = S.custom_scene(P, 4, seed=721, scale_lo=0.01, scale_hi=0.05)
    scene["centers"] *= spread
    scene["centers"][7::13] = 100.0  # behind or far off
    cams = S.make_cameras([(50 + 7 * (v % 3), 40) for v in range(views)], seed=722)
    rast = snp.Rasterizer(config_for(scene, persistent=1), P, cams)
    params = snp.params_to_device(scene)
    for away in (False, True):
        if away:  # nothing in any view
            params["centers"].fill_(1e4)
        inst = rast.prepare(params)
        keys, vals, _ = expected(rast)
        assert inst == len(keys)
        assert np.array_equal(rast.keys(inst).cpu().numpy().view(np.uint64), keys)
        assert np.array_equal(rast.values(inst).cpu().numpy().view(np.uint32), vals)
