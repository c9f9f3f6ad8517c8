"""The chain rule on either side of the set sizes and slice counts where its workgroups take
more Gaussians at a time, against the oracle's gradients.

Bars: within 1e-4 per parameter block, as in test_parity_render.py.
"""
import numpy as np
import pytest
import torch

from oracle import focus
from paper_2603_20611_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [33, 8128, 8192, 16384])
@pytest.mark.parametrize("slices", [1, 2, 3])
def test_gradients(gp, n, slices):
    from paper_2603_20611_amd import render as R
    print(f"[chain edges] n={n} slices={slices}", flush=True)
    p = synth.gaussians_uniform(n, (32.0, 24.0, 40.0), np.log(0.8), 0.2, seed=71)
    sl = synth.axial_slices(slices, 33, 23, 0.5, z0=19.0, dz=2.0)
    pt = torch.from_numpy(p).cuda()
    ws = R.Workspace()
    R.render(pt, sl, ws=ws)
    w = np.random.default_rng(9).standard_normal((slices, 23, 33)).astype(np.float32)
    g = R.render_backward(pt, sl, torch.from_numpy(w).cuda().reshape(-1), ws).cpu().numpy()
    want = focus.grad(p, sl, [x.astype(np.float64) for x in w])
    for r0, r1 in ((0, 3), (3, 6), (6, 10), (10, 11)):
        assert np.abs(g[r0:r1] - want[r0:r1]).max() <= 1e-4 * np.abs(want[r0:r1]).max()
    ws.close()
