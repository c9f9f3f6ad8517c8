"""The emit of mixed sigma_z from the codec's planes, in groups on both sides of the size
that leaves masks, against the oracle on the decoded set.

Bars: tile lists bit-exact, images within 1e-5 of the batch maximum, as in test_codec.py.
"""
import numpy as np
import pytest
import torch

from oracle import focus, quant, spec32
from paper_2603_20611_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns", [3, 32, 33])
def test_lists_and_images(gp, ns):
    from paper_2603_20611_amd import render as R
    print(f"[emit coded] ns={ns}", flush=True)
    n = 150
    p = synth.gaussians_uniform(n, (40.0, 36.0, 40.0), np.log(1.3), 0.3, seed=91)
    slices = synth.axial_slices(ns, 40, 36, 1.0, z0=0.3, dz=40.0 / ns)
    for k, s in enumerate(slices):
        s["sigma_z"] = (0.5, 3.0, 1.0, 0.0)[k % 4]
    codes, header, _ = R.encode(torch.from_numpy(np.ascontiguousarray(p)).cuda())
    d = quant.decode(codes.cpu().numpy().view(np.uint16)[:, :n], header.cpu().numpy())
    keys_ref, ranges_ref = spec32.bins(d, slices)
    ws = R.Workspace()
    out = R.render_coded(codes, header, n, slices, ws=ws).cpu().numpy()
    ws.check()
    keys, ranges = ws.export_bins(ranges_ref.shape[0], keys_ref.size + 16)
    assert np.array_equal(keys, keys_ref) and np.array_equal(ranges, ranges_ref)
    ref = np.concatenate([r.numpy().ravel() for r in focus.render(d, slices)])
    assert np.abs(out - ref).max() <= 1e-5 * np.abs(ref).max()
    ws.close()
