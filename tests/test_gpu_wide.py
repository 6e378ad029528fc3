"""Launches of few tiles give each 8 x 8 pixel block several waves.  The same
views rendered alone (four waves per block), with a further view that brings
the launch to three tiles per CU (two), and to seven (the plain kernels):
images equal bit for bit, gradients (the further view's loss gradient is zero)
to 1e-4 of the tensor's largest, float32 sums in no fixed order."""
import math

import numpy as np
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


def _render(scene, cams, cfg, pixels, dL):
    params = snp.params_to_device(scene)
    rast = snp.Rasterizer(cfg, len(scene["centers"]), cams)
    rast.prepare(params)
    images, T = rast.new_images()
    images.fill_(-1.0)
    rast.forward(params, images, T)
    counted, T2 = rast.new_images()
    rast.forward(params, counted, T2, count_pairs=True)  # always the plain kernel
    assert torch.equal(images, counted) and torch.equal(T, T2)
    rast.forward(params, images, T)  # the pair cache is this launch's
    full = torch.zeros_like(images)
    full[:3 * pixels] = dL
    grads = {k: torch.zeros_like(v) for k, v in params.items() if k != "opacity"}
    rast.backward(params, images, full, grads)
    return images[:3 * pixels].clone(), T[:pixels].clone(), grads


@pytest.mark.parametrize("N,fwd_cache,persistent,dense,options", [
    (4, 1, 0, False, {}), (8, 1, 1, True, {}), (16, 1, 0, True, {"alpha_max": 0.9}), (32, 1, 1, False, {}),
    (8, 0, 0, True, {"alpha_min": 1.0 / 255.0}), (32, 0, 1, True, {}), (16, 0, 0, False, {"t_eps": 0.0})])
def test_waves_per_block_by_the_number_of_tiles(N, fwd_cache, persistent, dense, options):
    # a dense scene ends pixels inside a batch; 230 primitives of 0.1 .. 0.4
    # give tiles more instances than a batch holds
    lo, hi = (0.1, 0.4) if dense else (0.02, 0.2)
    scene = S.custom_scene(230, N, seed=1011 + N, scale_lo=lo, scale_hi=hi)
    if dense:
        scene["w2"] = scene["w2"] * 8
    small = S.make_cameras([(75, 61), (33, 40)], seed=1012)
    pixels = 75 * 61 + 33 * 40
    cfg = config_for(scene, tile=(16, 16, 1), fwd_cache=fwd_cache, persistent=persistent, **options)
    dL = torch.from_numpy(np.random.default_rng(1013).normal(size=3 * pixels).astype(np.float32)).cuda() / pixels
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    want = None
    for per_cu in (7, 3, 0):
        cams = list(small)
        if per_cu:
            side = int(math.ceil(math.sqrt(per_cu * cus)))
            cams += S.make_cameras([(16 * side, 16 * side)], seed=1014)
            assert per_cu * cus <= side * side < (per_cu + 1) * cus - 40
        images, T, grads = _render(scene, cams, cfg, pixels, dL)
        if want is None:
            want = (images, T, grads)
            continue
        assert torch.equal(images, want[0]) and torch.equal(T, want[1])
        for k, g in grads.items():
            err, top = float((g - want[2][k]).abs().max()), float(want[2][k].abs().max())
            say(f"  {per_cu} tiles per CU, {k}: {err:.2e} of {top:.2e}")
            assert err <= 1e-4 * top
