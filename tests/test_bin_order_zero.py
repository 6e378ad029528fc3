"""bin_order 0 shows what the header says: with fewer than 2^16 (view,
primitive) pairs the layout, the instance offsets (a scan in primitive order)
and the counters of bin_order 2, from there on those of bin_order 1 (a scan in
the depth order of all pairs)."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2510_08491_amd as snp
import synthetic as S
from paper_2510_08491_amd import RenderConfig, _lib as L
from paper_2510_08491_amd.render import camera_array


@pytest.mark.parametrize("primitive", [0, 1])
@pytest.mark.parametrize("persistent", [0, 1])
@pytest.mark.parametrize("P,sizes", [
    (1, [(64, 64)]), (300, [(90, 70), (33, 40)]), (3000, [(320, 320)]), (16384, [(200, 117)] * 3),
    (16385, [(800, 800)] * 3), (65535, [(4112, 4096)]), (65536, [(90, 70)]), (15, [(33, 40)] * 4096)])
def test_layout(P, sizes, persistent, primitive):
    cams = camera_array(S.make_cameras(sizes, seed=1901))
    for cap in (1, 1000, 65536, 1 << 20):
        lays = []
        for order in (0, 1 if P * len(sizes) >= 1 << 16 else 2):
            cfg = RenderConfig(n_hidden=8, primitive=primitive, bin_order=order, persistent=persistent).to_c()
            lays.append(L.SnpLayout())
            assert L.lib().snp_workspace_layout(C.byref(cfg), P, len(sizes), cams, cap, C.byref(lays[-1])) == L.SNP_OK
        for f, _ in L.SnpLayout._fields_:
            assert getattr(lays[0], f) == getattr(lays[1], f), (cap, f)


@pytest.mark.gpu
@pytest.mark.parametrize("primitive", [0, 1])
@pytest.mark.parametrize("P,sizes", [(1, [(64, 64)]), (300, [(90, 70), (33, 40)]), (1025, [(50, 40)] * 7),
                                     (16384, [(90, 70)] * 3), (16385, [(90, 70)] * 3), (65535, [(90, 70)]),
                                     (65536, [(90, 70)])])
def test_offsets_and_counters(P, sizes, primitive):
    print(f"[gpu-test] {P} {len(sizes)} {primitive}", flush=True)
    scene = S.custom_scene(P, 4, seed=1902, scale_lo=0.01, scale_hi=0.05, primitive=primitive)
    scene["centers"][7::13] = 100.0  # behind or far off
    cams = S.make_cameras(sizes, seed=1903)
    params = snp.params_to_device(scene)
    pairs = P * len(sizes)
    lists = []
    for order in (0, 1, 2):
        rast = snp.Rasterizer(RenderConfig(n_hidden=4, omega0=float(scene["omega0"]), primitive=primitive,
                                           bin_order=order, fwd_cache=0), P, cams)
        inst = rast.prepare(params)
        counts = rast.tile_counts().cpu().numpy().ravel().astype(np.int64)
        depth = rast.depth_bits().cpu().numpy().ravel().view(np.uint32)
        offsets = rast._view("offsets", torch.int32, pairs).cpu().numpy().view(np.uint32)
        by_depth = order == 1 or (order == 0 and pairs >= 1 << 16)
        if not by_depth:
            assert np.array_equal(offsets, np.cumsum(counts) - counts)
        else:  # one depth order of all pairs, also of several views
            c = counts[np.argsort(depth, kind="stable")]
            assert np.array_equal(offsets, np.cumsum(c) - c)
        out = (C.c_int64 * 8)()
        L.check(L.lib().snp_read_counters(rast.ws_ptr, C.byref(rast.layout), out, None), "snp_read_counters")
        assert (out[0], out[1], out[7]) == (counts.sum(), 0, pairs if by_depth else 0)
        lists.append((rast.keys(inst).clone(), rast.values(inst).clone(), rast.ranges().clone()))
    for got in lists[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got, lists[0]))
