"""2^30 (view, primitive) pairs, where a launch of four threads per pair would
have the 2^32 threads that HIP refuses: all but 400 primitives lie behind every
camera, and the frame is the one of those 400 alone, bit for bit."""
import numpy as np
import pytest
import torch

import paper_2510_08491_amd as snp
import synthetic as S
from synthetic.scenes import look_at_camera
from tests.gpu_helpers import config_for, say

pytestmark = pytest.mark.gpu


def _frame(scene, params, cams, capacity):
    rast = snp.Rasterizer(config_for(scene, alpha_min=1.0 / 255.0), len(params["centers"]), cams, capacity=capacity)
    inst = rast.prepare(params, grow=False)
    images, T = rast.new_images()
    rast.forward(params, images, T)
    torch.cuda.synchronize()
    return inst, images, T


def test_four_threads_per_pair_at_2_to_the_30_pairs():
    say("[gpu-test] 2^30 pairs")
    P, V, seen = 1 << 20, 1024, 400
    free, _ = torch.cuda.mem_get_info()
    if free < 170 << 30:
        pytest.skip("needs 170 GiB of device memory")
    scene = S.custom_scene(seen, 8, color_mode=2, seed=1711, scale_lo=0.02, scale_hi=0.2, primitive=1)
    rng = np.random.default_rng(1712)
    cams = [look_at_camera(24, 20, np.append(rng.uniform(-0.5, 0.5, 2), -4.0)) for _ in range(V)]
    few = snp.params_to_device(scene)
    inst, images, T = _frame(scene, few, cams, 1 << 21)
    assert V * seen <= inst and float(T.min()) < 0.9
    many = {}
    for k, v in few.items():
        many[k] = v[:1].expand(P, *v.shape[1:]).clone()
        many[k][:seen // 2], many[k][-(seen // 2):] = v[:seen // 2], v[seen // 2:]
    many["centers"][seen // 2:-(seen // 2)] = torch.tensor([0.0, 0.0, -100.0], device="cuda")
    say(f"  {inst} instances of the 400 alone")
    inst2, images2, T2 = _frame(scene, many, cams, 1 << 21)
    assert inst2 == inst
    assert torch.equal(images2, images) and torch.equal(T2, T)
