"""Hundreds and thousands of views of few primitives: the instances of a host
sort whichever way their pairs are put in order, and no slower by default
(bin_order 0) than by the passes over all pairs (bin_order 1)."""
import numpy as np
import pytest
import torch

import paper_2510_08491_amd as snp
import synthetic as S
from tests.gpu_helpers import config_for, say
from tests.test_gpu_order import expected

pytestmark = pytest.mark.gpu


def _bin_us(rast):
    best = float("inf")
    x = torch.ones(4096, 4096, device="cuda")
    for _ in range(5):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        x @ x  # the launches are queued behind it
        a.record()
        for _ in range(10):
            rast.bin()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 100.0)
    return best


@pytest.mark.parametrize("V,P", [(511, 127), (512, 127), (513, 127), (1024, 63), (4096, 15)])
def test_views_of_few_primitives(V, P):
    say(f"[gpu-test] {V} views of {P}")
    scene = S.custom_scene(P, 4, seed=2101, scale_lo=0.02, scale_hi=0.1)
    cams = S.make_cameras([(24, 20)] * V, seed=2102)
    params = snp.params_to_device(scene)
    times = []
    for order in (0, 1):
        rast = snp.Rasterizer(config_for(scene, bin_order=order, fwd_cache=0), P, cams)
        inst = rast.prepare(params)
        keys, vals, _ = expected(rast)
        assert inst == len(keys)
        assert np.array_equal(rast.keys(inst).cpu().numpy().view(np.uint64), keys)
        assert np.array_equal(rast.values(inst).cpu().numpy().view(np.uint32), vals)
        times.append(_bin_us(rast))
    say(f"  bin: {times[0]:.0f}, {times[1]:.0f} us")
    assert times[0] <= 1.5 * times[1]
