"""The voxeliser's adjoint where tiles list more entries than one wavefront should sweep,
on grids of few and of many tiles, and its cost there.

Bars: gradients within 1e-4 of the oracle's per parameter block, as in
test_voxel_edges.py.  Time: the forward sweeps a tile's list with one wavefront; the
adjoint, about three times the arithmetic per entry, spread over more, must not
take longer than it.
"""
import numpy as np
import pytest
import torch

from oracle import voxel as ovox
from paper_2603_20611_amd import synth

pytestmark = pytest.mark.gpu

# name: (Gaussians in the clump, its edge, grid); twenty strays more.  On a grid of one
# tile all of them are in its list; else all of the clump in that of the tile at its middle.
LISTS = {f"list_{n}": (n - 20, 2.0, dict(nx=8, ny=8, nz=8)) for n in (63, 64, 65, 127, 128, 129)}
LISTS["list_777_65_tiles"] = (777, 6.0, dict(nx=37, ny=8, nz=103))
LISTS["list_500_ragged"] = (500, 5.0, dict(nx=75, ny=66, nz=41))


def _full(g):
    grid = dict(x0=0.0, y0=0.0, z0=0.0, dx=1.0, dy=1.0, dz=1.0)
    grid.update(g)
    return grid


@pytest.mark.parametrize("name", sorted(LISTS))
def test_gradients_of_long_lists(gp, name):
    from paper_2603_20611_amd import render as R
    n, side, g = LISTS[name]
    grid = _full(g)
    print(f"[voxel dense] {name}", flush=True)
    p = synth.gaussians_uniform(n, (side,) * 3, np.log(1.1), 0.3, seed=31)
    p[0:3] += 4.0 - side / 2
    strays = synth.gaussians_uniform(20, (float(grid["nx"]), float(grid["ny"]), float(grid["nz"])), 0.2, 0.2, seed=32)
    p = np.ascontiguousarray(np.concatenate([p, strays], axis=1))
    pt = torch.from_numpy(p).cuda()
    ws = R.Workspace()
    R.voxelize(pt, grid, ws)
    shape = (grid["nz"], grid["ny"], grid["nx"])
    w = np.random.default_rng(5).normal(size=shape).astype(np.float32)
    got = R.voxelize_backward(pt, grid, torch.from_numpy(w).cuda().reshape(-1), ws).cpu().numpy()
    want = ovox.grad(p, grid, w)
    for r0, r1 in ((0, 3), (3, 6), (6, 10), (10, 11)):
        assert np.abs(got[r0:r1] - want[r0:r1]).max() <= 1e-4 * np.abs(want[r0:r1]).max()
    ws.close()


def _best(f, reps=9):
    times = []
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        a.record()
        f()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b))
    return min(times[2:])


@pytest.mark.parametrize("name, n, side, edge", [("few_tiles", 100_000, 48.0, 48), ("clump", 100_000, 48.0, 256)])
def test_backward_of_long_lists_is_spread(gp, name, n, side, edge):
    from paper_2603_20611_amd import render as R
    print(f"[voxel dense] {name}", flush=True)
    grid = _full(dict(nx=edge, ny=edge, nz=edge))
    p = torch.from_numpy(synth.gaussians_uniform(n, (side,) * 3, np.log(1.5), 0.3, seed=33)).cuda()
    ws = R.Workspace()
    vol = torch.empty(edge ** 3, device="cuda")
    gvol = torch.rand(edge ** 3, device="cuda")
    grad = torch.zeros_like(p)
    fwd = _best(lambda: R.voxelize(p, grid, ws, out=vol))
    bwd = _best(lambda: R.voxelize_backward(p, grid, gvol, ws, grad=grad))
    print(f"   forward {fwd:.3f} ms, backward {bwd:.3f} ms", flush=True)
    assert bwd <= fwd
    ws.close()
