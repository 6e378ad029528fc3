"""Per-ray colour: chunks of the backward's gradient phase whose rows hold
different instances, whole and partial, against the FP64 oracle -- footprints
from one row to several chunks in random depth order."""
import pytest
import torch

import synthetic as S
from tests.gpu_helpers import config_for, grad_parity, say

pytestmark = pytest.mark.gpu

KEYS = ["centers", "scales", "quats", "w1", "b1", "w2", "b2", "colors", "cmlp"]


@pytest.fixture(autouse=True)
def _announce(request):
    say(f"[gpu-test] {request.node.name}")
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("N,fwd_cache,lo,hi", [(8, 1, 0.01, 0.03), (16, 0, 0.01, 0.5), (16, 1, 0.2, 0.6)])
def test_rows_of_different_instances(N, fwd_cache, lo, hi):
    scene = S.custom_scene(160, N, color_mode=4, cmlp_width=16, cmlp_depth=1, seed=1411 + N, scale_lo=lo, scale_hi=hi)
    cams = S.make_cameras([(75, 61), (33, 40)], seed=1312, lights=True)
    targets = S.make_targets(cams, seed=1313)
    grad_parity(scene, cams, targets, config_for(scene, tile=(16, 16, 1), fwd_cache=fwd_cache), KEYS)
