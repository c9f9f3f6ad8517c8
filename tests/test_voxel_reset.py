"""The voxeliser's reset of its tile ranges on grids of far more tiles than Gaussians.

Bits: the volume of a few Gaussians on a workspace that held a denser voxelisation is
that of a fresh workspace.  Time: the work is that of the tiles, so a few Gaussians may
not take a tenth longer than a thousand times as many.
"""
import pytest
import torch

from paper_2603_20611_amd import synth

pytestmark = pytest.mark.gpu


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


@pytest.mark.parametrize("edge", [1 << 13])
def test_few_gaussians_on_many_tiles(gp, edge):
    from paper_2603_20611_amd import render as R
    print("[voxel reset] few Gaussians on a million tiles", flush=True)
    grid = dict(nx=1, ny=edge, nz=edge)
    ws = R.Workspace()
    many = torch.from_numpy(synth.gaussians_uniform(65_536, (1.0, float(edge), float(edge)), 0.3, 0.2, seed=34)).cuda()
    vol = torch.empty(edge * edge, device="cuda")
    t_many = _best(lambda: R.voxelize(many, grid, ws, out=vol))
    few = many[:, :64].contiguous()
    t_few = _best(lambda: R.voxelize(few, grid, ws, out=vol))
    print(f"   65,536: {t_many:.3f} ms, 64: {t_few:.3f} ms", flush=True)
    w1 = R.Workspace()
    assert torch.equal(vol, R.voxelize(few, grid, w1))
    w1.close()
    assert t_few <= 1.1 * t_many
    ws.close()
