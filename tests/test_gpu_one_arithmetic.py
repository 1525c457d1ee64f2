"""One handle, one arithmetic: how a run is cut into calls, and whether its launches are
timed, changes no bit, also where the radial walls have no lanes of their own.

Handles whose step has no wall lanes by default: axis pipes of 64 k + 1 columns (their
wall column starts a wave), pipes of more than 1216 and annuli of more than 2496
columns (too few waves hold a wall).  Each runs in long calls (on tiles), in
calls of three steps and with timed launches (single steps), with the setting
at its default and switched either way, with checks inside the run.
"""
import numpy as np
import pytest

import lbm_inputs as li
from tests.test_gpu_batch import L, same  # noqa: F401
from tests.test_wall_lanes_host import _init

pytestmark = pytest.mark.gpu

CYLINDER = dict(r0=0.5, side_rmin="axis", side_rmax="wall", side_z="wall", therm_rmin="adiabatic",
                therm_rmax="fixed", therm_z="fixed", T_zmin=1.0, T_zmax=0.0, T_rmax=0.0, delta_T=1.0,
                T_ref=0.5, L=40.0, phi=0.7, Da=1e-2, F_phi=-1.0, Ra=1e4, Pr=0.7, nr=65, nz=60)
RATES = dict(s_j=1.3, s_q=0.9, s_e=1.4, s_eps=0.8, accel_r=2e-5, accel_z=1e-5)
CASES = {  # problem, porosity field, storage types, default setting
    "pipe 65x40": (li.pipe(nr=65, nz=40), False, ("fp32", "fp16", "bf16"), False),
    "pipe 129x50": (li.pipe(nr=129, nz=50), False, ("fp32", "fp16", "bf16"), False),
    "cylinder of 65 columns": (CYLINDER, False, ("fp32", "fp16", "bf16"), False),
    "developing pipe of 65 columns": (li.developing_pipe(Da=1e-2, nr=65, A=3.0, u_in=0.0025), False, ("fp32", "fp16"), False),
    "pipe 1300x24": (li.pipe(nr=1300, nz=24), False, ("fp32", "fp16"), False),
    "annulus 2530x33": (li.annulus(nr=2530, nz=33, Ra=1e5, Da=1e-3), False, ("fp32", "bf16"), False),
    "annulus 2600x40, porosity field": (li.annulus(nr=2600, nz=40, Ra=1e5, Da=1e-3), True, ("fp32", "fp16"), False),
    "annulus 65x70, other rates": (dict(li.annulus(nr=65, nz=70, Ra=1e5, Da=1e-3), **RATES), True,
                                   ("fp32", "fp16", "bf16"), True),
}


@pytest.mark.parametrize("mode", [-1, 0, 1])
@pytest.mark.parametrize("name,storage", [(n, s) for n in CASES for s in CASES[n][2]])
def test_calls_and_timing_change_no_bit(L, name, storage, mode):  # noqa: F811
    cfg, field, _, default = CASES[name]
    phi = [li.porosity_grf(cfg["nz"], cfg["nr"], seed=3)] if field else None
    init = [_init(cfg, 7)]
    run, one, timed = (L.Lattice([cfg], phi=phi, init=init, storage=storage, check_interval=50) for _ in range(3))
    for lat in (run, one, timed):
        assert lat.set_wall_lanes(mode) == (default if mode < 0 else bool(mode))
    timed.set_timing(True)
    for n in (6, 61, 53):
        run.step(n)
        timed.step(n)
        for _ in range(n // 3):
            one.step(3)
        one.step(n % 3)
        f = run.fields(0)
        assert np.isfinite(f["T"]).all() and np.isfinite(f["uz"]).all()
        same(f, one.fields(0), f"{name} {storage} mode {mode}, calls of three, {run.info()['t']} steps")
        same(f, timed.fields(0), f"{name} {storage} mode {mode}, timed, {run.info()['t']} steps")
    a, b = run.residual(), one.residual()
    for k in ("res", "nu_i", "nu_o", "status"):
        np.testing.assert_array_equal(a[k], b[k])
    assert run.step_paths()["tiles"] >= 100  # of 120
    assert one.step_paths()["tiles"] == timed.step_paths()["tiles"] == 0
    for lat in (run, one, timed):
        lat.close()
