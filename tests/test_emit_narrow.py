"""The emit of batches of one to eight slices, whose wavefronts take at least a round of
(Gaussian, slice) pairs: lists of a chunk below, at and above what one wavefront, or
four, take.

Bar: tile lists bit-exact against the binary32 specification.
"""
import numpy as np
import pytest
import torch

from oracle import spec32
from paper_2603_20611_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 64, 65, 257, 700])
@pytest.mark.parametrize("ns", [1, 2, 3, 8])
@pytest.mark.parametrize("fixed", [False, True])
def test_lists(gp, n, ns, fixed):
    from paper_2603_20611_amd import render as R
    print(f"[emit narrow] n={n} ns={ns} fixed={fixed}", flush=True)
    # a thin set: every Gaussian has a record on most of the slices
    p = synth.gaussians_uniform(n, (50.0, 40.0, 3.0), np.log(1.2), 0.3, seed=81)
    slices = synth.axial_slices(ns, 50, 40, 1.0, z0=0.2, dz=0.4)
    keys_ref, ranges_ref = spec32.bins(p, slices)
    ws = R.Workspace(capacity=(1 << 14, 1 << 17)) if fixed else R.Workspace()
    R.render(torch.from_numpy(np.ascontiguousarray(p)).cuda(), slices, ws=ws)
    ws.check()
    keys, ranges = ws.export_bins(ranges_ref.shape[0], keys_ref.size + 16)
    assert np.array_equal(keys, keys_ref) and np.array_equal(ranges, ranges_ref)
    ws.close()
