"""Folded Shack-Hartmann transform at the edges of its folds: every kind of
subaperture width (one pixel, odd with a middle sample, the widest), odd sample
counts (a frequency that is its own mirror image), an odd number of pixels
across (a pixel row that is its own pair) with even and odd rebin, focal planes
above 256 samples.  Bounds as for the other sensors (float32 sums of at most
32 + 32 terms against float64)."""

import numpy as np
import pytest

from oracle import sh as SH
from workloads import von_karman_opd

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,n,M,r", [
    (4, 4, 12, 3), (8, 4, 2, 1), (9, 3, 21, 7), (12, 4, 9, 9), (18, 3, 30, 6), (18, 2, 35, 5), (20, 2, 42, 6),
    (30, 2, 36, 12), (34, 2, 27, 3), (48, 2, 40, 8), (62, 2, 45, 9), (64, 2, 64, 4), (6, 2, 300, 12), (8, 2, 510, 34),
    (14, 2, 225, 15),
])
def test_fold_edges_match_oracle(D, n, M, r):
    from paper_2602_06688_amd import pwfs as P
    opd = von_karman_opd(range(2), D, 2.0, 0.3, 25.0, seed=D + M)
    print(f"[gpu] sh fold b={D // n} M={M} rebin={r}", flush=True)
    sh = P.SH(P.sh_desc(D, n, M, r, 0.0, 750.0), max_frames=2)
    sl, pix = sh.forward(torch.from_numpy(np.ascontiguousarray(opd, np.float32)).cuda(), want_pixels=True)
    torch.cuda.synchronize()
    want_pix, want_sl = SH.forward(opd.astype(np.float32).astype(np.float64), D, n, M, r, 0.0, 750.0)
    valid = SH.valid_subapertures(D, n, 0.0)   # the others' pixels are zero
    gp = pix.cpu().numpy()
    assert (gp[:, ~valid] == 0).all()
    assert np.abs(gp - want_pix)[:, valid].max() <= 1e-5 * np.abs(want_pix[:, valid]).max()
    assert np.abs(sl.cpu().numpy() - want_sl).max() <= 1e-5


@pytest.mark.parametrize("y,x", [(3, 3), (0, 6), (3, 1)])
def test_a_sample_that_is_not_finite_reaches_every_pixel_of_its_subaperture(y, x):
    from paper_2602_06688_amd import pwfs as P
    opd = torch.zeros(1, 28, 28, device="cuda")
    opd[0, 7 + y, 14 + x] = float("nan")
    sh = P.SH(P.sh_desc(28, 4, 60, 15, 0.0, 750.0), max_frames=1)
    sl, pix = sh.forward(opd, want_pixels=True)
    torch.cuda.synchronize()
    bad = torch.isnan(pix).flatten(3).sum(-1)[0].cpu().numpy()
    want = np.zeros((4, 4), int)
    want[1, 2] = 16
    assert (bad == want).all() and bool(torch.isfinite(sl).all())
