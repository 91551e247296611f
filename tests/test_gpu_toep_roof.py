"""Double roofs in the Toeplitz layouts at the edges of a column block (16 lines,
8-sample groups): the flat axis of either arm is copied between the layouts,
padding lines and samples left out, for every parity of 8-sample groups.  Bounds
as for the other FP32 sensors; a frame alone has the bits it has in a batch."""

import numpy as np
import pytest

import parity
from oracle import pwfs as O
from test_gpu_roof import _windows
from workloads import FLAG_DOUBLE_ROOF, FLAG_REF_SLOPES, tiny_sensor, von_karman_opd

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,N,sep,n_mod,lams,rings,frames", [
    (4, 64, 20, 2, (750.0,), 0, 3), (16, 64, 16, 5, (750.0,), 0, 40), (18, 64, 30, 8, (750.0, 900.0), 0, 9),
    (34, 128, 62, 7, (750.0,), 1, 5), (66, 256, 128, 16, (750.0,), 0, 30), (130, 384, 156, 6, (750.0, 900.0), 0, 4),
    (194, 512, 254, 6, (750.0,), 0, 4),
])
def test_flat_axes_at_block_edges(D, N, sep, n_mod, lams, rings, frames):
    from paper_2602_06688_amd import pwfs as P
    s = tiny_sensor(n_pupil=D, n_fft=N, n_subap=max(2, D // 4), pupil_sep_px=float(sep), n_mod=n_mod, mod_radius_lod=2.0,
                    lambdas_nm=lams, lambda_weights=(1.0 / len(lams),) * len(lams), lambda_ref_nm=750.0,
                    src_rings=rings, src_radius_lod=1.0 if rings else 0.0, flags=FLAG_DOUBLE_ROOF | FLAG_REF_SLOPES)
    pick = [0, frames - 1]
    opd = np.zeros((frames, D, D), np.float32)
    opd[pick] = von_karman_opd(range(2), D, s.diameter_m, 0.3, 25.0, seed=D)
    opd[1:-1] = opd[0] * np.linspace(0.1, 0.9, frames - 2, dtype=np.float32)[:, None, None]
    x = torch.from_numpy(opd).cuda()
    print(f"[gpu] toeplitz roof D={D} N={N} n_mod={n_mod} lambdas={len(lams)} rings={rings} frames={frames}", flush=True)
    plan = P.Plan([s], max_frames=frames)
    I, sl, _ = plan.step(x)
    one = [plan.step(x[f:f + 1].contiguous()) for f in pick]
    torch.cuda.synchronize()
    W = _windows(I.cpu().numpy().reshape(frames, 2, N, N), s)
    assert all(np.array_equal(W[f], _windows(o[0].cpu().numpy().reshape(1, 2, N, N), s)[0]) for f, o in zip(pick, one))
    I_ref = O.forward(opd[pick].astype(np.float64), s)
    s_ref, _ = O.slopes(I_ref, s)
    err = parity.errors(W[pick].astype(np.float64), _windows(I_ref, s), sl.cpu().numpy()[pick].astype(np.float64), s_ref,
                        O.valid_subapertures(s))
    print(f"      {parity.fmt(err)}", flush=True)
    parity.check(err, parity.FP32)
