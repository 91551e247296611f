"""The three forms of the Toeplitz column pass (whole, split over workgroups,
half-split) give a frame the same bits, for every number of 32-sample steps, on
both sides of a step's edges, with groups of unequal size and two wavelengths;
the bits are within the FP32 bounds of the FP64 oracle.  Which form a number of
frames takes is checked on the host (test_host_routes.py)."""

import numpy as np
import pytest

import parity
from oracle import pwfs as O
from workloads import tiny_sensor, von_karman_opd

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# pupil, grid, separation, points, wavelengths; frames of the half-split, split and whole form (0: not taken)
CASES = [
    (32, 64, 32, 12, 1, 0, 3, 50), (34, 128, 62, 9, 1, 14, 0, 15), (64, 128, 64, 16, 1, 6, 7, 31),
    (66, 256, 128, 16, 1, 5, 6, 21), (94, 256, 126, 6, 2, 5, 6, 15), (98, 256, 126, 7, 1, 9, 10, 12),
    (128, 256, 128, 9, 1, 5, 6, 11), (130, 384, 156, 6, 2, 3, 4, 15), (160, 512, 192, 7, 1, 6, 7, 13), (160, 512, 192, 5, 1, 6, 7, 9),
    (162, 384, 192, 6, 1, 5, 6, 12), (192, 384, 192, 16, 1, 2, 3, 13), (194, 512, 254, 7, 1, 4, 5, 10),
    (222, 512, 254, 6, 2, 2, 3, 10), (226, 768, 384, 6, 1, 4, 5, 9), (256, 768, 384, 7, 1, 4, 5, 9),
]


def sensor(D, N, sep, n_mod, nl):
    lams = (750.0, 900.0)[:nl]
    return tiny_sensor(n_pupil=D, n_fft=N, n_subap=D // 4, pupil_sep_px=float(sep), n_mod=n_mod, mod_radius_lod=3.0,
                       obstruction=0.1, lambdas_nm=lams, lambda_weights=(0.625, 0.375) if nl == 2 else (1.0,),
                       lambda_ref_nm=750.0)


def _windows(I, s):
    D = s.n_pupil
    return np.stack([I[:, r:r + D, c:c + D] for r, c in O.image_origins(s)], axis=1)


@pytest.mark.parametrize("D,N,sep,n_mod,nl,half,split,whole", CASES)
def test_forms_give_the_same_bits(D, N, sep, n_mod, nl, half, split, whole):
    from paper_2602_06688_amd import pwfs as P
    s = sensor(D, N, sep, n_mod, nl)
    opd = np.zeros((whole, D, D), np.float32)
    opd[0] = von_karman_opd(1, D, s.diameter_m, 0.15, 25.0, seed=D)[0]
    opd[1:] = opd[0] * np.linspace(0.1, 0.9, whole - 1, dtype=np.float32)[:, None, None]
    x = torch.from_numpy(opd).cuda()
    print(f"[gpu] toeplitz forms D={D} N={N} n_mod={n_mod} lambdas={nl} frames {half} {split} {whole}", flush=True)
    plan = P.Plan([s], max_frames=whole)
    I, sl, _ = [t.clone() for t in plan.step(x)]
    W = _windows(I.cpu().numpy(), s)
    assert np.isfinite(W).all()
    for few in (f for f in (1, half, split) if f):
        Wf = _windows(plan.step(x[:few].contiguous())[0].cpu().numpy(), s)
        assert np.array_equal(Wf, W[:few]), few
    I_ref = O.forward(opd[:1], s)
    s_ref, _ = O.slopes(I_ref, s)
    err = parity.errors(W[:1].astype(np.float64), _windows(I_ref, s), sl.cpu().numpy()[:1].astype(np.float64), s_ref,
                        O.valid_subapertures(s))
    print(f"      {parity.fmt(err)}", flush=True)
    parity.check(err, parity.FP32)
