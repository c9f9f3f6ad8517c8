"""The bin ranges of small sorts: of one pass (the digit is the bin) and of two, with many
pairs on few bins and with bins that stay empty.

Bits: lists and ranges against the binary32 specification.  Time: the sort of the same
Gaussians by 64 bins (one pass) may not take longer than by 1,024 (two).
"""
import numpy as np
import pytest
import torch

from oracle import spec32
from paper_2603_20611_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width, height", [(16, 16), (33, 16), (128, 128), (129, 240), (350, 340), (360, 350), (500, 512)])
@pytest.mark.parametrize("n", [1, 700, 30_000])
def test_lists(gp, width, height, n):
    from paper_2603_20611_amd import render as R
    print(f"[sort ranges] {width} x {height} n={n}", flush=True)
    # the Gaussians on half of the slice: the other bins stay empty
    p = synth.gaussians_uniform(n, (width / 2, float(height), 4.0), np.log(0.7), 0.2, seed=61)
    sl = synth.axial_slices(1, width, height, 3.0, z0=2.0)
    keys_ref, ranges_ref = spec32.bins(p, sl)
    ws = R.Workspace()
    pt = torch.from_numpy(np.ascontiguousarray(p)).cuda()
    for _ in range(2):   # the second render meets the first one's ranges
        R.render(pt, sl, ws=ws)
    keys, ranges = ws.export_bins(ranges_ref.shape[0], keys_ref.size + 16)
    assert np.array_equal(keys, keys_ref) and np.array_equal(ranges, ranges_ref)
    ws.close()


def test_few_bins_are_not_slower(gp):
    from paper_2603_20611_amd import render as R
    ms = []
    for edge in (128, 512):
        p = synth.gaussians_uniform(1_000_000, (float(edge), float(edge), 4.0), np.log(0.5), 0.2, seed=62)
        pt = torch.from_numpy(np.ascontiguousarray(p)).cuda()
        sl = synth.axial_slices(1, edge, edge, 3.0, z0=2.0)
        ws = R.Workspace()
        R.render(pt, sl, ws=ws)
        best = 1e9
        for _ in range(8):
            ws.set_timing(True, ["sort"])
            R.render(pt, sl, ws=ws)
            best = min(best, ws.timings()["sort"][0])
        ms.append(best)
        ws.close()
    print(f"[sort ranges] 64 bins {ms[0]:.4f} ms, 1,024 bins {ms[1]:.4f} ms", flush=True)
    assert ms[0] <= ms[1]
