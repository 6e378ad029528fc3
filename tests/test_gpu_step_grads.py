"""A step stores its gradients, the backward entry adds them: a step into
buffers full of NaN gives what the backward adds to zeros, for every colour
mode, also when only some gradients are asked for; and repeated persistent
launches on one workspace (whose queue the launch itself puts back) give the
same images.  Gradients are float32 sums in no fixed order: equal to 1e-4 of
the tensor's largest."""
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


@pytest.mark.parametrize("color_mode,persistent,some,temporal", [
    (0, 1, None, False), (1, 1, None, False), (2, 0, None, False), (2, 1, None, True), (3, 1, None, False),
    (4, 1, None, False), (3, 0, ["centers", "w2"], False), (4, 0, ["centers"], False), (1, 1, ["cmlp"], False),
    (2, 1, ["sh", "quats"], False)])
def test_step_stores_what_the_backward_adds(color_mode, persistent, some, temporal):
    width = 16 if color_mode in (1, 3, 4) else 0
    scene = S.custom_scene(140, 8, color_mode=color_mode, cmlp_width=width, cmlp_depth=1, seed=911, scale_lo=0.05,
                           scale_hi=0.3)
    rng = np.random.default_rng(912)
    if temporal:
        scene["wt"] = rng.uniform(-3, 3, (140, 8)).astype(np.float32)
        scene["sh_t"] = rng.uniform(-0.3, 0.3, (140, 12, 3)).astype(np.float32)
    scene["centers"][:9] += 50.0  # seen by no view
    cams = S.make_cameras([(70, 60), (41, 52)], seed=913, lights=True)
    cfg = config_for(scene, tile=(16, 16, 1), persistent=persistent)
    params = snp.params_to_device(scene)
    rast = snp.Rasterizer(cfg, 140, cams)
    rast.prepare(params)
    images, T = rast.new_images()
    tg = torch.from_numpy(np.concatenate([t.ravel() for t in S.make_targets(cams, seed=914)]).astype(np.float32)).cuda()
    keys = [k for k in params if k != "opacity" and (some is None or k in some)]  # (no gradient: Gaussians only)
    want = {k: torch.zeros_like(params[k]) for k in keys}
    rast.forward(params, images, T)
    loss, dL = rast.loss_l1(images, tg)
    rast.backward(params, images, dL, want)
    first = images.clone()
    n = float(3 * rast.total_pixels)
    for _ in range(3):
        got = {k: torch.full_like(params[k], float("nan")) for k in keys}
        images.fill_(-1.0)
        rast.step(params, images, T, tg, n, loss, dL, got)
        assert torch.equal(images, first)
        images.fill_(-1.0)
        rast.forward(params, images, T)
        assert torch.equal(images, first)
        for k in keys:
            err = float((got[k] - want[k]).abs().max())
            say(f"  {k}: {err:.2e} of {float(want[k].abs().max()):.2e}")
            assert err <= 1e-4 * float(want[k].abs().max())
