"""The autotuner times only settings that change what a plan runs: no row tile for
sensors whose row pass has none, one launch schedule per pass size.  CPU."""

import pytest

import host_routes
from paper_2602_06688_amd import autotune as A
from paper_2602_06688_amd import pwfs as P
from test_autotune import FakePlan, _sensor as fake_sensor
from workloads import FLAG_DOUBLE_ROOF, FLAG_FULL_PLANE, PREC_BF16, PREC_FP16X3, tiny_sensor


def _sensor(D, N, n_mod=8, **kw):
    return tiny_sensor(n_pupil=D, n_fft=N, n_subap=D // 4, pupil_sep_px=float(min(N - D, 2 * (D * 3 // 5))), n_mod=n_mod,
                       mod_radius_lod=2.0, **kw)


# sensor, whether its row pass has a tile
SENSORS = [
    (_sensor(80, 256), False), (_sensor(256, 768), False), (_sensor(258, 768), True), (_sensor(64, 128), False),
    (_sensor(80, 256, fov_lod=30.0), True), (_sensor(80, 256, flags=FLAG_FULL_PLANE), True),
    (_sensor(80, 256, flags=FLAG_DOUBLE_ROOF), False), (_sensor(80, 256, flags=FLAG_DOUBLE_ROOF, fov_lod=30.0), True),
    (_sensor(226, 512, n_mod=15), False), (_sensor(226, 512, n_mod=16), True), (_sensor(224, 512, n_mod=48), False),
    (_sensor(256, 512, n_mod=3, src_rings=1, src_radius_lod=1.0), True), (_sensor(256, 768, n_mod=48), False),
    (_sensor(226, 512, n_mod=48, flags=FLAG_DOUBLE_ROOF), False),
    (_sensor(226, 512, n_mod=48, precision=PREC_FP16X3), False),
    (_sensor(80, 256, precision=PREC_FP16X3), False), (_sensor(80, 256, precision=PREC_BF16), False),
]


def test_row_tile_rule_is_the_library_s_route():
    exe = host_routes.build()
    if exe is None:
        pytest.skip("hipcc or the built library not available")
    host = host_routes.Host(exe)
    for s, tiled in SENSORS:
        assert P.takes_row_tile(s) is tiled
        assert host.plan([s], 2)[0] == 0
        rc, launches = host.forward(2)
        host.free()
        assert rc == 0 and any(x[0] == "k_rows" for x in launches) is tiled
    host.close()


def test_tiles_are_tried_on_the_sensors_that_have_them(tmp_path):
    class Plan(FakePlan):
        def takes_row_tile(self, i):
            return i in (1, 3)
    sens = [fake_sensor(160, 512), fake_sensor(160, 512), fake_sensor(80, 256), fake_sensor(240, 768)]
    plan = Plan(sens)
    rec = A.autotune(plan, lambda: None, 10, cache_path=str(tmp_path / "c.json"), timer=lambda: 1.0)
    tried = {tuple(t["row_tiles"]) for t in rec["tried"] if any(t["row_tiles"])}
    assert tried == {(0, 16, 0, 0), (0, 0, 0, 16)}


def test_one_launch_schedule_per_pass_size():
    plan = FakePlan()
    launches = [c for c in A.candidates(plan) if c["mode"] == P.MODE_LAUNCHES]
    assert sorted(c["chunk"] for c in launches) == [6, 13, 26]
    assert {(c["wg_per_cu"], c["row_groups"]) for c in launches} == {(2, 2048)}
