"""The float64 autograd route where a unit's phase hardly changes along the
chord (a scene in which one pair's phase gradient vanishes but for 1e-8): its
gradients against central differences of the numpy renderer's loss, to the 1e-3
that the kernels' gradients are held to."""
import numpy as np
import pytest

import synthetic as S
from oracle.grad import autograd_loss_and_grads, numpy_loss
from oracle.render import RenderOptions

OPTS = RenderOptions()


@pytest.fixture(scope="module")
def scene():
    sc = S.custom_scene(160, 16, seed=1327, scale_lo=0.01, scale_hi=0.5)
    cams = S.make_cameras([(75, 61), (33, 40)], seed=1312, lights=True)
    tg = S.make_targets(cams, seed=1313)
    return sc, cams, tg, autograd_loss_and_grads(sc, cams, tg, OPTS)[1]


@pytest.mark.parametrize("axis", [0, 1, 2])
def test_gradient_of_a_unit_with_a_flat_phase(scene, axis):
    sc, cams, tg, grads = scene
    vals = []
    for sgn in (1.0, -1.0):
        w1 = np.asarray(sc["w1"], dtype=np.float64).copy()
        w1[61, 14, axis] += sgn * 1e-3
        vals.append(numpy_loss({**sc, "w1": w1}, cams, tg, OPTS))
    fd = (vals[0] - vals[1]) / 2e-3
    got = grads["w1"][61, 14, axis]
    print(f"autograd {got:.6e}, central difference {fd:.6e}")
    assert abs(got - fd) <= 1e-3 * abs(fd)
