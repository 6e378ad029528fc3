"""The autograd entry lets the kernels set its gradients in fresh memory: every
element set, whatever the memory held, zero for a parameter that the colour
mode does not use, against the accumulating entry into zeros (float32 sums in
no fixed order: 1e-4 of the tensor's largest)."""
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


@pytest.mark.parametrize("color_mode,extra", [(0, "sh"), (0, "xi"), (1, "colors"), (2, "sh_t"), (3, None), (4, "xi")])
def test_gradients_in_fresh_memory(color_mode, extra):
    P = 130
    width = 16 if color_mode in (1, 3, 4) else 0
    scene = S.custom_scene(P, 8, color_mode=color_mode, cmlp_width=width, cmlp_depth=1, seed=1111, scale_lo=0.05,
                           scale_hi=0.3)
    scene["centers"][:9] += 50.0  # seen by no view
    if extra:
        shape = {"sh": (P, 16, 3), "xi": (P, 8), "colors": (P, 3), "sh_t": (P, 12, 3)}[extra]
        scene[extra] = np.random.default_rng(1112).normal(size=shape).astype(np.float32)
    scene.pop("opacity", None)
    cams = S.make_cameras([(70, 60), (41, 52)], seed=1113, lights=True)
    rast = snp.Rasterizer(config_for(scene, tile=(16, 16, 1)), P, cams)
    params = {k: v.requires_grad_(True) for k, v in snp.params_to_device(scene).items()}
    dL = torch.randn(3 * rast.total_pixels, device="cuda") / rast.total_pixels
    for _ in range(2):
        for v in params.values():
            v.grad = None
        images, T = snp.splat_render(rast, params)
        junk = [torch.full_like(v, float("nan")) for v in params.values() for _ in range(3)]
        del junk  # what the allocator hands out next
        images.backward(dL)
        want = snp.zeros_like_params({k: v.detach() for k, v in params.items()})
        rast.backward({k: v.detach() for k, v in params.items()}, images.detach(), dL, want)
        for k, v in params.items():
            err, top = float((v.grad - want[k]).abs().max()), float(want[k].abs().max())
            say(f"  {k}: {err:.2e} of {top:.2e}")
            assert err <= 1e-4 * top
        if extra and not (color_mode == 2 and extra == "sh_t"):
            assert not params[extra].grad.any()
