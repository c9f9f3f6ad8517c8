"""The two loss terms of batches of thousands of workgroups, whose sums the first workgroup
of the gradient adds up, for maps below and above the size where its first pass
changes, against a float64 evaluation on the device.

Bar: 1e-6, a few binary32 roundings of the float64 sums (the result is binary32, and
added to a zero).
"""
import numpy as np
import pytest
import torch

from oracle import ssim as ossim

pytestmark = pytest.mark.gpu


def _filter(img, w):
    """The separable window over [s, h, w] images, zeros outside."""
    r = (len(w) - 1) // 2
    for dim in (1, 2):
        n = img.shape[dim]
        pad = torch.nn.functional.pad(img, (0, 0, r, r) if dim == 1 else (r, r, 0, 0))
        img = sum(float(c) * pad.narrow(dim, k, n) for k, c in enumerate(w))
    return img


@pytest.mark.parametrize("s, h, w", [(1000, 17, 33), (40, 256, 256), (11, 1017, 1003), (23, 500, 977)])
def test_loss_terms(gp, s, h, w):
    from paper_2603_20611_amd import render as R
    print(f"[ssim sums] {(s, h, w)}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(8)
    x = torch.rand(s, h, w, device="cuda", generator=gen)
    y = torch.rand(s, h, w, device="cuda", generator=gen)
    ws = R.Workspace()
    loss = torch.zeros(2, device="cuda")
    R.l1_dssim_loss_grad(x.reshape(-1), y.reshape(-1), s, w, h, ws, lam=0.2, loss=loss)
    win = np.asarray(ossim.window(), np.float64)
    win = win.sum(0) if win.ndim == 2 else win
    xd, yd = x.double(), y.double()
    mx, my = _filter(xd, win), _filter(yd, win)
    vx, vy, c = _filter(xd * xd, win) - mx * mx, _filter(yd * yd, win) - my * my, _filter(xd * yd, win) - mx * my
    S = (2 * mx * my + 1e-4) * (2 * c + 9e-4) / ((mx * mx + my * my + 1e-4) * (vx + vy + 9e-4))
    want = [(xd - yd).abs().mean().item(), (1.0 - S).mean().item()]
    got = loss.cpu().numpy().astype(np.float64)
    for a, b in zip(got, want):
        assert abs(a - b) <= 1e-6 * abs(b)
    ws.close()
