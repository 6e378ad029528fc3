"""Binning at the sizes where its kernels change: pairs ordered by one
workgroup (up to 16384) or by radix passes with blocks of 1024 or 4096 keys,
one to three passes over the instances, ties in depth, culled pairs, empty
views, and the full-key sort (bin_order 2) -- keys, values, ranges and the
prefix sums against a host sort of the same pairs, bit for bit."""
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


def expected(rast):
    """Sorted (keys, values) of the workspace's rectangles and depths."""
    rects = rast.rects().cpu().numpy().astype(np.int64)
    depth = rast.depth_bits().cpu().numpy().view(np.uint32).astype(np.uint64)
    counts = rast.tile_counts().cpu().numpy().view(np.uint32)
    tw, th = rast.cfg.tile_w, rast.cfg.tile_h
    keys, vals, base = [], [], 0
    for v, c in enumerate(rast.cams):
        nx, ny = -(-c.width // tw), -(-c.height // th)
        for p in np.nonzero(counts[v])[0]:
            x0, x1, y0, y1 = rects[v, p]
            ty, tx = np.meshgrid(np.arange(y0 // th, y1 // th + 1), np.arange(x0 // tw, x1 // tw + 1), indexing="ij")
            t = (base + ty * nx + tx).ravel().astype(np.uint64)
            assert len(t) == counts[v, p]
            keys.append((t << np.uint64(31)) | depth[v, p])
            vals.append(np.full(len(t), p, np.uint32))
        base += nx * ny
    keys = np.concatenate(keys) if keys else np.zeros(0, np.uint64)
    vals = np.concatenate(vals) if vals else np.zeros(0, np.uint32)
    order = np.argsort(keys, kind="stable")  # ties keep the (view, primitive) order
    return keys[order], vals[order], base


@pytest.mark.parametrize("P,sizes,bin_order,primitive", [
    (1, [(64, 64)], 0, 0), (63, [(64, 64)], 0, 1), (1025, [(95, 61)], 0, 0), (8192, [(160, 90), (80, 80)], 0, 0),
    (16385, [(200, 117)], 0, 0), (16385, [(200, 117)], 1, 1), (16385, [(200, 117)], 2, 0),
    (70000, [(96, 64), (1, 1), (61, 33), (96, 64)], 0, 0), (30000, [(1600, 1300), (1600, 1300)], 0, 0),
    (300, [(4096, 2304)], 0, 0)])
def test_sorted_instances_match_a_host_sort(P, sizes, bin_order, primitive):
    scene = S.custom_scene(P, 8, seed=701, scale_lo=0.01, scale_hi=0.06, primitive=primitive)
    # equal depths (duplicates) and primitives behind the camera
    scene["centers"][1::3] = scene["centers"][0::3][:len(scene["centers"][1::3])]
    scene["centers"][5::11] *= 40.0
    cams = S.make_cameras(sizes, seed=702)
    cfg = config_for(scene, bin_order=bin_order, persistent=1)
    rast = snp.Rasterizer(cfg, P, cams)
    params = snp.params_to_device(scene)
    for _ in range(2):  # the second time over a used workspace
        inst = rast.prepare(params)
        keys, vals, tiles = expected(rast)
        assert inst == len(keys)
        assert np.array_equal(rast.keys(inst).cpu().numpy().view(np.uint64), keys)
        assert np.array_equal(rast.values(inst).cpu().numpy().view(np.uint32), vals)
        tile = (keys >> np.uint64(31)).astype(np.int64)
        start = np.searchsorted(tile, np.arange(tiles), "left")
        end = np.searchsorted(tile, np.arange(tiles), "right")
        ranges = rast.ranges().cpu().numpy().view(np.uint32).astype(np.int64)
        full = end > start
        assert np.array_equal(ranges[full], np.stack([start, end], 1)[full]) and not ranges[~full].any()
        images, T = rast.new_images()  # every tile is taken once
        images.fill_(-1.0)
        rast.forward(params, images, T)
        assert float(images.min()) >= 0.0
