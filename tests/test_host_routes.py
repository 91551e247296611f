"""Which launches a plan makes, and that they stay inside its scratch: host code
of the built library alone (tests/host_routes.py), no GPU."""

import time

import pytest

import host_routes
from test_gpu_toep_forms import CASES as FORMS, sensor as forms_sensor
from workloads import FLAG_DOUBLE_ROOF, FLAG_REF_SLOPES, PREC_BF16X3, PREC_FP16X3, PREC_FP32, tiny_sensor


@pytest.fixture(scope="module")
def host():
    exe = host_routes.build()
    if exe is None:
        pytest.skip("hipcc or the built library not available")
    h = host_routes.Host(exe)
    yield h
    h.close()


def _sensor(D, N, sep, n_mod, nl=1, prec=PREC_FP32, flags=0, rings=0):
    lams = tuple(750.0 + 10.0 * i for i in range(nl))
    return tiny_sensor(n_pupil=D, n_fft=N, n_subap=max(1, D // 4), pupil_sep_px=float(sep), n_mod=n_mod, mod_radius_lod=3.0,
                       lambdas_nm=lams, lambda_weights=(1.0 / nl,) * nl, lambda_ref_nm=750.0, precision=prec,
                       flags=flags, src_rings=rings, src_radius_lod=1.0 if rings else 0.0)


# sensor, frames, and the pass size that plans of the FFT and dense forms accept
# for it: 12 GiB of their scratch per pass
PASSES = [
    (_sensor(136, 512, 336, 73, rings=2), 454, 92),
    (_sensor(6, 128, 82, 820, nl=15, prec=PREC_FP16X3), 917, 917),
    (_sensor(120, 512, 176, 828, prec=PREC_BF16X3), 350, 126),
    (_sensor(244, 768, 250, 637), 986, 40),
    (_sensor(54, 768, 364, 857, flags=FLAG_DOUBLE_ROOF), 551, 542),
    (_sensor(62, 128, 64, 89, nl=10), 770, 446),
    (_sensor(180, 512, 238, 37, nl=14, flags=FLAG_DOUBLE_ROOF | FLAG_REF_SLOPES), 493, 85),
    (_sensor(234, 768, 250, 91, prec=PREC_FP16X3, flags=FLAG_REF_SLOPES), 979, 308),
]


@pytest.mark.parametrize("i", range(len(PASSES)))
def test_pass_sizes_of_saved_tunings_stay_accepted(host, i):
    """A tuning saved with the pass size that a sensor's FFT or dense form accepts
    is accepted by the Toeplitz form too, whose scratch takes more per frame; its
    passes are then as large as the scratch holds."""
    s, frames, accepted = PASSES[i]
    rc, most, _ = host.plan([s], frames)
    assert rc == 0
    try:
        assert most >= accepted
        rc, _, chunk = host.tune(0, accepted)
        assert rc == 0 and chunk == accepted
        rc, launches = host.forward(frames)
        assert rc == 0
        rows = [x for x in launches if x[0] in ("k_toep_rows", "k_toep_cols", "k_toep_cols_halves")]
        assert rows and all(x[3] == 0 for x in rows)
    finally:
        host.free()


PWFS_EWORKSPACE = -3


@pytest.mark.parametrize("s", [_sensor(160, 512, 192, 48), _sensor(64, 128, 64, 16), _sensor(30, 64, 34, 7, nl=2),
                               _sensor(160, 512, 192, 48, flags=FLAG_DOUBLE_ROOF), _sensor(256, 768, 384, 7, nl=3),
                               _sensor(96, 256, 120, 16, rings=1, flags=FLAG_REF_SLOPES)],
                         ids=["160", "64", "30", "roof", "256", "source"])
def test_every_pass_stays_in_its_scratch_and_a_smaller_one_is_refused(host, s):
    """Row output and unit sums of every pass size end inside the sensor's scratch
    (with few frames the sums lie behind them); a scratch that does not hold them
    is refused before anything is launched."""
    frames = 48
    assert host.plan([s], frames)[0] == 0
    try:
        parts = set()
        for nf in range(1, frames + 1):
            rc, launches = host.forward(nf)
            assert rc == 0
            passes = [x for x in launches if x[0] in ("k_toep_rows", "k_toep_cols", "k_toep_cols_halves")]
            assert passes and all(x[3] == 0 for x in passes), (nf, passes)
            parts |= {x[2] > 1 for x in passes if x[0] != "k_toep_rows"}
        assert True in parts
        size, seen = host.scratch(0), set()
        for k in range(41):
            host.scratch(0, size * k // 40 - host.scratch(0))
            for nf in (1, frames):
                rc, launches = host.forward(nf)
                seen.add(rc)
                assert all(not x[3] for x in launches)
                if rc and not s.flags & FLAG_DOUBLE_ROOF:      # a roof's first arm may fit where its second does not
                    assert not launches
        assert seen == {0, PWFS_EWORKSPACE}
    finally:
        host.free()


@pytest.mark.parametrize("rings", [0, 1, 2, 8])
@pytest.mark.parametrize("n_mod", [1, 2, 3, 4, 15, 16])
def test_points_are_counted_as_they_are_listed(host, n_mod, rings):
    assert host.plan([_sensor(20, 64, 20, n_mod, rings=rings)], 1)[0] == 0
    n_pts, n_keys, pts, keys = host.points()
    host.free()
    assert (n_pts, n_keys) == (pts, keys)


def test_sizing_a_plan_does_not_list_its_points():
    """The layout needs the numbers of points and x-tilts dozens of times: sizing
    4096 points took 8.7 ms where each was a sorted list, 8 us for 4."""
    from paper_2602_06688_amd import pwfs as P

    def best(s):
        ts = []
        for _ in range(7):
            t = time.perf_counter()
            P.workspace_size([s], 1)
            ts.append(time.perf_counter() - t)
        return min(ts)
    assert best(_sensor(20, 64, 20, 4096)) < 10 * best(_sensor(20, 64, 20, 4))


@pytest.mark.parametrize("i", range(len(FORMS)))
def test_frames_of_the_forms_test_take_their_forms(host, i):
    D, N, sep, n_mod, nl, half, split, whole = FORMS[i]
    assert host.plan([forms_sensor(D, N, sep, n_mod, nl)], whole)[0] == 0
    try:
        for frames, form in ((half, "half"), (split, "split"), (whole, "whole")):
            if frames:
                rc, launches = host.forward(frames)
                (cols,) = [x for x in launches if x[0] in ("k_toep_cols", "k_toep_cols_halves")]
                sums = [x for x in launches if x[0] == "k_toep_sum"]
                assert rc == 0 and cols[3] == 0
                assert (cols[0] == "k_toep_cols_halves", cols[2] > 1, len(sums)) == {
                    "half": (True, True, 1), "split": (False, True, 1), "whole": (False, False, 0)}[form]
    finally:
        host.free()
