"""Gradients against the FP64 oracle in scenes where a unit's phase hardly
changes along a pair's chord (phase gradients down to 1e-9)."""
import math

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


def test_per_ray_colour():
    scene = S.custom_scene(160, 16, color_mode=4, cmlp_width=16, cmlp_depth=1, seed=1327, scale_lo=0.01, scale_hi=0.5)
    cams = S.make_cameras([(75, 61), (33, 40)], seed=1312, lights=True)
    grad_parity(scene, cams, S.make_targets(cams, seed=1313), config_for(scene, tile=(16, 16, 1), fwd_cache=0),
                KEYS + ["cmlp"])


def test_few_tiles():
    scene = S.custom_scene(120, 16, seed=1527, scale_lo=0.02, scale_hi=0.15)
    side = 16 * (int(math.sqrt(4 * torch.cuda.get_device_properties(0).multi_processor_count)) - 1) + 1
    cams = S.make_cameras([(side, side)], seed=1512)
    grad_parity(scene, cams, S.make_targets(cams, seed=1513), config_for(scene, tile=(16, 16, 1), fwd_cache=0), KEYS)
