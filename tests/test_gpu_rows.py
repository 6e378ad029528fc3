"""The backward's gradient phase packs the live pairs of a batch into rows of
16 of one instance: footprints from part of a row to several chunks of 64,
mixed within a batch, every density width and every backward batch size,
against the FP64 oracle's gradients."""
import numpy as np
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


@pytest.mark.parametrize("N,tile,fwd_cache", [
    (4, (16, 16, 1, 8), 1), (8, (16, 16, 1, 4), 1), (8, (16, 16, 1, 16), 0), (16, (16, 16, 1, 8), 0),
    (32, (16, 16, 1, 4), 1), (8, (8, 8, 1, 32), 1), (16, (8, 8, 1, 16), 1), (8, (32, 16, 2, 8), 1)])
def test_rows_of_small_and_large_footprints(N, tile, fwd_cache):
    # scales 0.008 .. 0.5 at 55 pixels per unit distance: 1 to a few thousand
    # pixels per primitive, in random depth order
    scene = S.custom_scene(220, N, seed=611, scale_lo=0.008, scale_hi=0.5)
    cams = S.make_cameras([(95, 61), (33, 40)], seed=612)
    targets = S.make_targets(cams, seed=613)
    cfg = config_for(scene, tile=tile, fwd_cache=fwd_cache)
    grad_parity(scene, cams, targets, cfg, KEYS)
