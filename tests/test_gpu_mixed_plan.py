"""Plans that hold FFT sensors (behind a field stop, or wider than 256 pixels) and
Toeplitz sensors side by side, and the FFT passes of window sensors: the
persistent mode makes one launch for each kind, whose counters lie apart and
whose error flag is shared.  Both modes against each other and the FP64 oracle."""

import numpy as np
import pytest

import parity
from oracle import pwfs as O
from test_gpu_hetero import _packed, _unpack, _windows
from workloads import PREC_BF16X3, PREC_FP16X3, PREC_FP32, tiny_sensor, von_karman_opd

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TWO = dict(lambdas_nm=(700.0, 900.0), lambda_weights=(0.5, 0.5), lambda_ref_nm=700.0)


def _sensor(D, N, n_mod, fov=0.0, n_subap=0, **kw):
    return tiny_sensor(n_pupil=D, n_fft=N, n_subap=n_subap or D // 4, n_mod=n_mod, pupil_sep_px=float(2 * (D * 3 // 5)),
                       mod_radius_lod=2.0, obstruction=0.2, diameter_m=8.0, fov_lod=fov, **kw)


def _mixed():
    """FFT, Toeplitz, FFT, Toeplitz, ...: D, N, points, stop"""
    return [_sensor(80, 256, 8, 25.0), _sensor(96, 256, 6), _sensor(160, 512, 4, 30.0), _sensor(120, 384, 5, **TWO),
            _sensor(264, 768, 3, n_subap=33), _sensor(240, 768, 4), _sensor(100, 384, 4, 20.0, **TWO)]


def _inputs(sensors, F):
    opds = [von_karman_opd(F, s.n_pupil, 8.0, 0.3, 25.0, seed=60 + i) for i, s in enumerate(sensors)]
    return opds, torch.from_numpy(_packed(opds)).cuda()


def _against_oracle(plan, opds, I, S, frames=slice(None)):
    Is = _unpack(plan, I.cpu().numpy().astype(np.float64), "I")
    Ss = _unpack(plan, S.cpu().numpy().astype(np.float64), "S")
    for s, o, Ig, Sg in zip(plan.sensors, opds, Is, Ss):
        I_ref = O.forward(o[frames], s)
        s_ref, _ = O.slopes(I_ref, s)
        err = parity.errors(_windows(Ig[frames], s), _windows(I_ref, s), Sg[frames], s_ref, O.valid_subapertures(s))
        print(f"      D={s.n_pupil} N={s.n_fft}: {parity.fmt(err)}", flush=True)
        parity.check(err, parity.FP32)


def test_persistent_equals_launches_and_oracle():
    from paper_2602_06688_amd import pwfs as P
    sensors, F = _mixed(), 3
    opds, x = _inputs(sensors, F)
    plan = P.Plan(sensors, max_frames=F)
    print("[gpu] mixed plan: launches", flush=True)
    I0, S0, F0 = [t.clone() for t in plan.step(x)]
    _against_oracle(plan, opds, I0, S0, slice(0, 1))
    for chunk in (1, 3):
        for w in (1, 3):
            print(f"[gpu] mixed plan: persistent chunk={chunk} wg_per_cu={w}", flush=True)
            plan.set_tuning(mode=P.MODE_PERSISTENT, chunk=chunk, wg_per_cu=w)
            I1, S1, F1 = plan.step(x)
            plan.status()
            assert torch.equal(I0, I1) and torch.equal(S0, S1) and torch.equal(F0, F1)


@pytest.mark.parametrize("order", [(0, 1, 2, 3), (0, 2, 6), (1, 3, 5)], ids=["mixed", "fft", "toeplitz"])
def test_waits_that_give_up_are_reported_for_either_kind(order):
    """Forced from the host (a negative spin limit): every waiting item is skipped,
    the launches end, the status says so once, and the plan runs again."""
    from paper_2602_06688_amd import pwfs as P
    sensors = [_mixed()[i] for i in order]
    _, x = _inputs(sensors, 2)
    plan = P.Plan(sensors, max_frames=2)
    I0, S0, _ = [t.clone() for t in plan.step(x)]
    plan.status()
    print(f"[gpu] plan {order}: every dependency wait forced to give up", flush=True)
    plan.set_tuning(mode=P.MODE_PERSISTENT, spin_limit=-1)
    plan.forward(x)
    with pytest.raises(P.PwfsError) as ei:
        plan.status()
    assert ei.value.code == P.PWFS_EHIP and "gave up" in str(ei.value)
    plan.status()
    plan.set_tuning(spin_limit=0)
    I1, S1, _ = plan.step(x)
    plan.status()
    assert torch.equal(I0, I1) and torch.equal(S0, S1)


def test_row_tiles_of_the_fft_passes_give_identical_bits_in_both_modes():
    from paper_2602_06688_amd import pwfs as P
    sensors = [_sensor(80, 256, 8, 25.0), _sensor(120, 384, 4, 30.0, **TWO), _sensor(160, 512, 4, 30.0),
               _sensor(240, 768, 3, 40.0), _sensor(264, 768, 3, n_subap=33)]
    opds, x = _inputs(sensors, 2)
    plan = P.Plan(sensors, max_frames=2)
    assert all(plan.takes_row_tile(i) for i in range(5))
    assert [plan.row_tile(i) for i in range(5)] == [8, 16, 8, 8, 8]
    I0, S0, _ = [t.clone() for t in plan.step(x)]
    _against_oracle(plan, opds, I0, S0, slice(0, 1))
    alt = [16, 8, 16, 16, 16]
    for mode in (P.MODE_LAUNCHES, P.MODE_PERSISTENT):
        for pick in ([1, 1, 1, 1, 1], [0, 1, 0, 1, 0]):
            tiles = [a if p else 0 for a, p in zip(alt, pick)]
            print(f"[gpu] fft passes: mode {mode} row tiles {tiles}", flush=True)
            for i, r in enumerate(tiles):
                plan.set_row_tile(i, r)
            plan.set_tuning(mode=mode)
            I1, S1, _ = plan.step(x)
            plan.status()
            assert torch.equal(I0, I1) and torch.equal(S0, S1)


@pytest.mark.parametrize("D,N,n_mod,sep,prec", [
    (226, 512, 16, 270, PREC_FP32), (256, 512, 17, 256, PREC_FP32), (258, 768, 3, 300, PREC_FP32),
    (300, 768, 4, 360, PREC_FP32), (258, 768, 3, 300, PREC_FP16X3), (258, 768, 3, 300, PREC_BF16X3),
    (300, 768, 2, 360, PREC_BF16X3),
])
def test_windows_that_are_not_toeplitz_products_match_oracle(D, N, n_mod, sep, prec):
    """On both sides of the width from which the FFT and dense forms take the windows."""
    from paper_2602_06688_amd import pwfs as P
    s = tiny_sensor(n_pupil=D, n_fft=N, n_subap=D // 6, pupil_sep_px=float(sep), n_mod=n_mod, mod_radius_lod=3.0,
                    obstruction=0.1, precision=prec)
    opd = von_karman_opd(2, D, s.diameter_m, 0.15, 25.0, seed=D)
    print(f"[gpu] wide windows D={D} N={N} n_mod={n_mod} precision={prec}", flush=True)
    plan = P.Plan([s], max_frames=2)
    I, sl, _ = plan.step(torch.from_numpy(np.ascontiguousarray(opd, np.float32)).cuda())
    torch.cuda.synchronize()
    ref = s.with_(precision=PREC_FP32)
    I_ref = O.forward(opd, ref)
    s_ref, _ = O.slopes(I_ref, ref)
    err = parity.errors(_windows(I.cpu().numpy().astype(np.float64), s), _windows(I_ref, s),
                        sl.cpu().numpy().astype(np.float64), s_ref, O.valid_subapertures(s))
    print(f"      {parity.fmt(err)}", flush=True)
    parity.check(err, {PREC_FP32: parity.FP32, PREC_FP16X3: parity.FP16X3, PREC_BF16X3: parity.BF16X3}[prec])
