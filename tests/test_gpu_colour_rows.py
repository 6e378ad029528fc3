"""The colour network's adjoint keeps LDS rows for four or for sixteen views
of a chunk: view counts around both, with primitives that some chunk, or every
view, does not see, every width and depth, against the FP64 oracle."""
import pytest
import torch

import synthetic as S
from tests.gpu_helpers import config_for, grad_parity, say

pytestmark = pytest.mark.gpu

KEYS = ["centers", "scales", "quats", "w1", "b1", "w2", "b2", "cmlp", "xi"]


@pytest.fixture(autouse=True)
def _announce(request):
    say(f"[gpu-test] {request.node.name}")
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("views,width,depth,color_mode", [
    (1, 16, 3, 1), (3, 32, 1, 1), (4, 32, 3, 3), (5, 16, 1, 3), (16, 32, 2, 1), (18, 16, 2, 1)])
def test_view_counts_around_the_rows(views, width, depth, color_mode):
    scene = S.custom_scene(70, 8, color_mode=color_mode, cmlp_width=width, cmlp_depth=depth, seed=811 + views,
                           scale_lo=0.05, scale_hi=0.3)
    # ten primitives far outside every view, five behind part of the cameras
    scene["centers"][:10] += 40.0
    scene["centers"][10:15] *= 4.0
    cams = S.make_cameras([(30 + v, 26) for v in range(views)], seed=812, lights=True)
    targets = S.make_targets(cams, seed=813)
    cfg = config_for(scene, tile=(16, 16, 1))
    grad_parity(scene, cams, targets, cfg, KEYS + (["colors"] if color_mode == 3 else []))
