"""The order of the tiles where several workgroups make it (more than 5120
tiles): every tile once, also when all or most of them are empty, which does
not make them wait for each other."""
import pytest
import torch

import paper_2510_08491_amd as snp
import synthetic as S
from tests.gpu_helpers import config_for, say

pytestmark = pytest.mark.gpu


def _sort_us(rast):
    best = float("inf")
    x = torch.ones(4096, 4096, device="cuda")
    for _ in range(5):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        x @ x  # the sorts are queued behind it
        a.record()
        for _ in range(10):
            rast.sort()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 100.0)
    return best


@pytest.mark.parametrize("P,scale,sides", [(1, 1e-3, (70, 190)), (300, 0.1, (71, 72)), (3000, 0.2, (70, 75))])
def test_many_tiles(P, scale, sides):
    say(f"[gpu-test] {P} primitives of {scale}")
    scene = S.custom_scene(P, 4, seed=2001, scale_lo=scale, scale_hi=scale)
    params = snp.params_to_device(scene)
    cams = S.make_cameras([(1120, 1120)], seed=2002)
    want, times = None, []
    for side in (0,) + sides:  # 4900 tiles, then with a further view of side x side
        more = S.make_cameras([(16 * side - 15, 16 * side)], seed=2003) if side else []
        rast = snp.Rasterizer(config_for(scene, persistent=1, fwd_cache=0), P, cams + more)
        assert rast.layout.total_tiles == 4900 + side * side
        rast.prepare(params)
        images, T = rast.new_images()
        images.fill_(-1.0)
        rast.forward(params, images, T)
        times.append(_sort_us(rast))
        assert float(images.min()) >= 0.0  # no tile left out
        one = images[:3 * 1120 * 1120].clone()
        want = one if want is None else want
        assert torch.equal(one, want)
    say("  sort: " + ", ".join(f"{t:.0f}" for t in times) + " us")
    if P == 1:  # 41000 empty tiles: 340 us where each waited for the one before
        assert times[2] <= 4.0 * times[0]
