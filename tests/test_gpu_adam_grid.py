"""The optimizer's launch at the edges of its grid (2048 workgroups of 256
parameters), against the float64 oracle: one pass of the grid less or more by
one parameter, group edges inside a later pass, several passes with a rest."""
import numpy as np
import pytest
import torch

from oracle import train as T
from paper_2510_08491_amd import train as TR
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu

GRID = 2048 * 256


@pytest.mark.parametrize("sizes", [(GRID - 1,), (GRID,), (GRID - 1, 2), (3, GRID, 1, GRID + 5), (2 * GRID + 77, 1, GRID)])
def test_adam_at_the_edges_of_its_grid(sizes):
    say(f"[gpu-test] {sizes}")
    rng = np.random.default_rng(len(sizes) + sum(sizes))
    keys = ["centers", "scales", "quats", "w1"][:len(sizes)]
    host = {k: np.exp(rng.uniform(-4, 0, n)).astype(np.float32) for k, n in zip(keys, sizes)}
    dev = {k: torch.from_numpy(p.copy()).cuda() for k, p in host.items()}
    opt = TR.Adam(dev)
    ref = {k: (p.astype(np.float64), np.zeros(p.shape), np.zeros(p.shape)) for k, p in host.items()}
    for step in (1, 2):
        grads = {k: (rng.standard_normal(p.shape) * 1e-3).astype(np.float32) for k, p in host.items()}
        opt.step({k: torch.from_numpy(g).cuda() for k, g in grads.items()})
        for k in keys:
            p, m, v = ref[k]
            ref[k] = T.adam_step(p, grads[k].astype(np.float64), m, v, step, TR.PAPER_LRS[k],
                                 log_space=(k == "scales"))
    torch.cuda.synchronize()
    for k in keys:
        p, m, v = ref[k]
        # tolerances of the optimizer's parity test: the value to 2e-6, the step to 1e-5 of the
        # rate (|m_hat| <= 2 sqrt(v_hat) here, a few roundings of 6e-8), moments normwise to 1e-5
        err = np.max(np.abs(dev[k].cpu().numpy() - p) / (2e-6 * np.abs(p) + 1e-5 * TR.PAPER_LRS[k]))
        merr = np.max(np.abs(opt.m[k].cpu().numpy() - m)) / (1e-5 * np.max(np.abs(m)))
        verr = np.max(np.abs(opt.v[k].cpu().numpy() - v)) / (1e-5 * np.max(np.abs(v)))
        assert err <= 1 and merr <= 1 and verr <= 1, (k, err, merr, verr)
