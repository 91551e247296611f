"""Real-Toeplitz form of the image-window sensors against the FP64 oracle, at
the edges of its tiles (16 lines, 8-sample groups, 32-sample steps): the
smallest pupil, one sample pair past a tile, exactly full tiles, and the
largest one, with point counts around the summation groups (1, 2, 3, 7, 48)
and one to three wavelengths.

Bounds are the FP32 form's (tests/parity.py): the products carry 22
significand bits per operand with float32 sums, and the 1/2 z term is float32.
A lost product of the split errs near 1e-3.

``frames`` fills the chip, so a batch runs the column pass whole and one frame
alone runs it split over workgroups; both add in the same order and must give
the same bits, whatever else is in the batch (a frame of NaN)."""

import numpy as np
import pytest

import parity
from oracle import pwfs as O
from workloads import PREC_BF16X3, PREC_FP16X3, PREC_FP32, tiny_sensor, von_karman_opd

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BOUNDS = {PREC_FP32: parity.FP32, PREC_FP16X3: parity.FP16X3, PREC_BF16X3: parity.BF16X3}


def _windows(I, s):
    D = s.n_pupil
    return np.stack([I[:, r:r + D, c:c + D] for r, c in O.image_origins(s)], axis=1)


@pytest.mark.parametrize("D,N,sep,n_mod,lams,frames,prec", [
    (4, 64, 32, 3, (2200.0,), 1100, PREC_FP32),
    (30, 64, 34, 7, (2200.0, 1600.0), 1100, PREC_FP32),
    (32, 128, 64, 1, (2200.0,), 1100, PREC_FP32),
    (34, 128, 62, 48, (2200.0, 1600.0, 1250.0), 400, PREC_FP32),
    (66, 256, 128, 2, (2200.0,), 140, PREC_FP32),
    (98, 256, 126, 7, (2200.0,), 80, PREC_FP16X3),
    (128, 256, 128, 3, (2200.0,), 70, PREC_BF16X3),
    (158, 384, 190, 48, (2200.0,), 60, PREC_FP32),
    (160, 512, 256, 7, (2200.0, 1600.0), 56, PREC_FP32),
    (162, 384, 192, 3, (2200.0,), 26, PREC_FP32),
    (194, 512, 254, 7, (2200.0,), 22, PREC_FP32),
    (256, 768, 384, 7, (2200.0, 1250.0), 20, PREC_FP32),
])
def test_tile_edges_against_oracle_and_split_equals_whole(D, N, sep, n_mod, lams, frames, prec):
    from paper_2602_06688_amd import pwfs as P
    w = {1: (1.0,), 2: (0.625, 0.375), 3: (0.5, 0.3125, 0.1875)}[len(lams)]
    s = tiny_sensor(n_pupil=D, n_fft=N, n_subap=max(2, D // 4), pupil_sep_px=float(sep), n_mod=n_mod,
                    mod_radius_lod=3.0, obstruction=0.1, lambdas_nm=lams, lambda_weights=w,
                    lambda_ref_nm=lams[0], precision=prec)
    pick = [0, frames - 1]
    opd = np.zeros((frames, D, D), np.float32)
    opd[pick] = von_karman_opd(range(2), D, s.diameter_m, 0.15, 25.0, seed=D)
    opd[1:-1] = opd[0] * np.linspace(0.1, 0.9, frames - 2, dtype=np.float32)[:, None, None]
    opd[frames // 2] = np.nan
    x = torch.from_numpy(opd).cuda()
    print(f"[gpu] toeplitz form D={D} N={N} n_mod={n_mod} lambdas={len(lams)} frames={frames}", flush=True)
    plan = P.Plan([s], max_frames=frames)
    I, sl, _ = plan.step(x)
    one = [plan.step(x[f:f + 1].contiguous()) for f in pick]
    torch.cuda.synchronize()
    W = _windows(I.cpu().numpy(), s)
    assert all(np.array_equal(W[f:f + 1], _windows(o[0].cpu().numpy(), s)) for f, o in zip(pick, one))
    keep = np.arange(frames) != frames // 2
    assert np.isfinite(W[keep]).all() and np.isnan(W[~keep]).all()
    ref = s.with_(precision=PREC_FP32)
    I_ref = O.forward(opd[pick], ref)
    s_ref, _ = O.slopes(I_ref, ref)
    err = parity.errors(W[pick].astype(np.float64), _windows(I_ref, s), sl.cpu().numpy()[pick].astype(np.float64), s_ref,
                        O.valid_subapertures(s))
    print(f"      {parity.fmt(err)}", flush=True)
    parity.check(err, BOUNDS[prec])
