"""The workspace never shrinks as its instance capacity grows (the search for
the largest capacity that fits the static scratch bisects on that): capacities
around half the number of tiles, where the place of the tile order changes, and
around those where the sort's block size does.  And the tile order in spare keys that the tiles, not
the instances, give their size."""
import ctypes as C

import pytest
import torch

import paper_2510_08491_amd as snp
import synthetic as S
from paper_2510_08491_amd import RenderConfig, _lib as L
from paper_2510_08491_amd.render import camera_array


@pytest.mark.parametrize("persistent", [0, 1])
@pytest.mark.parametrize("bin_order", [0, 1, 2])
@pytest.mark.parametrize("sizes,P", [([(800, 800)], 300), ([(4096, 4096)], 64), ([(90, 70), (33, 40)], 20000),
                                     ([(4112, 4096)], 7), ([(600, 400)] * 3, 40000)])
def test_size_grows_with_capacity(sizes, P, bin_order, persistent):
    cams = camera_array(S.make_cameras(sizes, seed=1801))
    tiles = sum(-(-w // 16) * -(-h // 16) for w, h in sizes)
    caps = {c + d for c in (1, tiles // 2, tiles, P, 1 << 10, 1 << 12, 1 << 18, 1 << 20) for d in range(-3, 4)}
    last = 0
    for cap in sorted(c for c in caps if c > 0):
        lay = L.SnpLayout()
        cfg = RenderConfig(n_hidden=4, bin_order=bin_order, persistent=persistent, fwd_cache=0).to_c()
        assert L.lib().snp_workspace_layout(C.byref(cfg), P, len(sizes), cams, cap, C.byref(lay)) == L.SNP_OK
        assert lay.bytes >= last, (cap, last, lay.bytes)
        last = lay.bytes


@pytest.mark.gpu
@pytest.mark.parametrize("primitive,P", [(0, 40), (1, 12)])  # 266 and 622 instances
def test_more_tiles_than_room_for_their_order(primitive, P):
    print(f"[gpu-test] primitive {primitive}", flush=True)
    scene = S.custom_scene(P, 8, seed=1802, scale_lo=0.02, scale_hi=0.1, primitive=primitive)
    cams = S.make_cameras([(800, 800)], seed=1803)
    params = snp.params_to_device(scene)
    want = None
    for persistent in (0, 1):
        rast = snp.Rasterizer(RenderConfig(n_hidden=8, omega0=float(scene["omega0"]), primitive=primitive,
                                           persistent=persistent), P, cams, capacity=1200)
        inst = rast.prepare(params, grow=False)
        assert 200 < inst <= 1200 and rast.layout.total_tiles == 2500
        for _ in range(2):  # the sort's input stays in place
            rast.sort()
            images, T = rast.new_images()
            rast.forward(params, images, T)
            got = (rast.keys(inst).clone(), rast.values(inst).clone(), rast.ranges().clone(), images, T)
            want = want or got
            assert all(torch.equal(a, b) for a, b in zip(got, want))
