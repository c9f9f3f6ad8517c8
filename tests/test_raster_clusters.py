"""The backward rasteriser where most tiles are empty and a few list very many entries.

Time: the same clump on a grid just below and just above the bin count from which a
tile's list starts on one wavefront; the sweep of the clump is the same work, so the
stage may not take half as long again.  Bits: every list entry's moments are summed
alone, so the gradients of the two are equal.
"""
import numpy as np
import pytest
import torch

from paper_2603_20611_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, side", [(20_000, 32.0), (20_000, 64.0), (200_000, 64.0)])
def test_clump_on_large_grids(gp, n, side):
    from paper_2603_20611_amd import render as R
    print(f"[raster clusters] n={n} side={side}", flush=True)
    p = torch.from_numpy(synth.gaussians_uniform(n, (side, side, 32.0), np.log(1.5), 0.3, seed=51)).cuda()
    grads, ms = [], []
    for edge in (880, 1024):           # 12,100 and 16,384 bins
        sl = synth.axial_slices(4, edge, edge, 1.0, z0=4.1, dz=8.0)
        ws = R.Workspace()
        out = R.render(p, sl, ws=ws)
        g = torch.zeros(4, edge, edge, device="cuda")
        g[:, :100, :100] = torch.rand(4, 100, 100, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
        g = g.reshape(-1)
        grads.append(R.render_backward(p, sl, g, ws))
        best = 1e9
        scratch = torch.zeros_like(p)
        for _ in range(8):
            ws.set_timing(True, ["raster_bwd"])
            R.render_backward(p, sl, g, ws, grad=scratch)
            best = min(best, ws.timings()["raster_bwd"][0])
        ms.append(best)
        ws.close()
        del out
    print(f"   {ms[0]:.4f} ms, {ms[1]:.4f} ms", flush=True)
    assert torch.equal(grads[0], grads[1])
    assert ms[1] <= 1.5 * ms[0]
