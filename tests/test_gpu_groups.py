"""Kernels that give a group of lanes to each primitive (density table, per-ray
colour table, both adjoints): primitive counts around a workgroup's 64 and
view counts around its four waves, every density width, against the FP64
oracle's gradients."""
import pytest
import torch

import synthetic as S
from tests.gpu_helpers import config_for, grad_parity, say

pytestmark = pytest.mark.gpu

KEYS = ["centers", "scales", "quats", "w1", "b1", "w2", "b2", "colors"]


@pytest.fixture(autouse=True)
def _announce(request):
    say(f"[gpu-test] {request.node.name}")
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("P,N,views,color_mode", [
    (1, 4, 1, 0), (63, 8, 4, 0), (64, 16, 5, 0), (65, 32, 3, 0), (130, 4, 9, 0),
    (65, 16, 5, 4), (3, 8, 1, 4), (129, 8, 6, 2), (66, 16, 5, 1)])
def test_gradients_at_the_edges_of_the_groups(P, N, views, color_mode):
    width = 16 if color_mode in (1, 4) else 0
    scene = S.custom_scene(P, N, color_mode=color_mode, cmlp_width=width, cmlp_depth=1, seed=711 + P, scale_lo=0.05,
                           scale_hi=0.4)
    cams = S.make_cameras([(33 + v, 28) for v in range(views)], seed=712, lights=True)
    targets = S.make_targets(cams, seed=713)
    cfg = config_for(scene, tile=(16, 16, 1))
    keys = KEYS[:-1] + {0: ["colors"], 1: ["cmlp", "xi"], 2: ["sh"], 4: ["colors", "cmlp"]}[color_mode]
    grad_parity(scene, cams, targets, cfg, keys)
