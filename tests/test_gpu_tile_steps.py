"""Plain steps taken several at a time on LDS tiles against single steps on the GPU.

A handle whose calls are long runs on tiles; one stepped in calls of one to three
steps, and one that times its launches, takes single steps.  Every operation is
the same, so fields, residual and Nusselt numbers are bit-identical, in every
storage type, for grids of one tile, of ragged tiles and batches, with every
side condition, with checks inside the run, after compaction and after a
storage conversion.
"""
import numpy as np
import pytest

import lbm_inputs as li
from tests.test_gpu_batch import L, same  # noqa: F401
from tests.test_wall_lanes_host import _init

pytestmark = pytest.mark.gpu

CASES = {
    "pipe 64x8": ([li.pipe()], False),
    "pipe 40x70": ([li.pipe(nr=40, nz=70)], False),
    "annulus 5x4": ([li.annulus(nr=5, nz=4, Ra=1e4, Da=1e-2)], False),
    "annulus 33x24": ([li.annulus(nr=33, nz=24, Ra=1e4, Da=1e-2)], False),
    "annulus 65x130, porosity field": ([li.annulus(nr=65, nz=130, Ra=1e5, Da=1e-3)], True),
    "annulus 257x300": ([li.annulus(nr=257, nz=300, Ra=1e5, Da=1e-3)], False),
    "annulus 600x650, porosity field": ([li.annulus(nr=600, nz=650, Ra=1e6, Da=1e-3)], True),
    "periodic ends": ([dict(li.annulus(nr=90, nz=100, Ra=1e4, Da=1e-2), side_z="periodic", accel_z=1e-4)], False),
    "printed source": ([dict(li.annulus(nr=50, nz=61, Ra=1e5, Da=1e-3), src_printed=1)], False),
    "heater": ([li.heater_annulus(1e-2, nr=80, nz=90)], False),
    "inlet and outlet": ([li.developing_pipe(Da=1e-2, nr=41, A=8.0, u_in=0.0025)], False),
    "closed cylinder": ([dict(r0=0.5, side_rmin="axis", side_rmax="wall", side_z="wall", therm_rmin="adiabatic",
                              therm_rmax="fixed", therm_z="fixed", T_zmin=1.0, T_zmax=0.0, T_rmax=0.0, delta_T=1.0,
                              T_ref=0.5, L=40.0, phi=0.7, Da=1e-2, F_phi=-1.0, Ra=1e4, Pr=0.7, nr=41, nz=60)], False),
    "batch": (li.sweep(n_inst=9, sizes=[32, 64, 96]), False),
}


@pytest.mark.parametrize("storage", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("name", CASES)
def test_runs_on_tiles_equal_single_steps(L, name, storage):  # noqa: F811
    cfgs, field = CASES[name]
    phi = [li.porosity_grf(c["nz"], c["nr"], seed=3) for c in cfgs] if field else None
    init = [_init(c, 7) for c in cfgs]
    run = L.Lattice(cfgs, phi=phi, init=init, storage=storage, check_interval=50)
    one = L.Lattice(cfgs, phi=phi, init=init, storage=storage, check_interval=50)
    timed = L.Lattice(cfgs, phi=phi, init=init, storage=storage, check_interval=50)
    timed.set_timing(True)
    for n in (6, 61, 33, 100):  # even and odd starts, a check inside
        run.step(n)
        timed.step(n)
        for _ in range(n // 3):
            one.step(3)
        one.step(n % 3)
        for i in range(len(cfgs)):
            same(run.fields(i), one.fields(i), f"{name} {storage} instance {i}, {run.info()['t']} steps")
            same(run.fields(i), timed.fields(i), f"{name} {storage} timed, instance {i}")
    a, b = run.residual(), one.residual()
    for k in ("res", "nu_i", "nu_o", "status"):
        np.testing.assert_array_equal(a[k], b[k])
    for lat in (run, one, timed):
        lat.close()


def test_tiles_follow_compaction_and_storage_conversion(L):  # noqa: F811
    quiet = li.annulus(nr=64, nz=64, Ra=1e4, Da=1e-3)
    quiet.update(tol=10.0)  # converges at its first check
    cfgs = [li.annulus(nr=96, nz=72, Ra=1e5, Da=1e-3), quiet, li.annulus(nr=33, nz=97, Ra=1e6, Da=1e-2)]
    run, one = (L.Lattice(cfgs, storage="fp16", check_interval=20) for _ in range(2))
    for n in (61, 40):
        run.step(n)
        for _ in range(n):
            one.step(1)
        assert run.compact() == one.compact() == 2
    run.set_storage("fp32")
    one.set_storage("fp32")
    run.step(39)
    for _ in range(39):
        one.step(1)
    for i in range(3):
        a, b = run.info(i), one.info(i)
        a.pop("device_bytes"), b.pop("device_bytes")  # single steps keep no second set of planes
        assert a == b
        same(run.fields(i), one.fields(i), f"instance {i}")
    run.close()
    one.close()


@pytest.mark.parametrize("nr,nz", [(2600, 40), (3001, 33)])
def test_wide_grids_take_tiles_within_rounding(L, nr, nz):  # noqa: F811
    """Rows of more than 2560 columns: single steps leave the radial walls to their
    owners, tiles give them lanes.  The two differ by FP32 rounding (2e-6 of a
    field's norm, the bound between the two kernels of single steps), and a
    handle whose wall lanes are switched off takes single steps only."""
    c = li.annulus(nr=nr, nz=nz, Ra=1e5, Da=1e-3)
    init = [_init(c, 5)]
    got = []
    for mode, timed in ((-1, False), (-1, True), (0, False)):
        lat = L.Lattice([c], init=init, check_interval=0)
        lat.set_wall_lanes(mode)
        lat.set_timing(timed)
        lat.step(60)
        got.append(lat.fields(0))
        lat.close()
    same(got[1], got[2], "without wall lanes")
    for k in ("uz", "ur", "T"):
        a, b = got[0][k].astype(np.float64), got[1][k].astype(np.float64)
        assert np.linalg.norm(a - b) <= 2e-6 * np.linalg.norm(b), k


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
def test_fields_of_a_stopped_instance_are_those_of_its_own_level(L, storage):  # noqa: F811
    """An instance that stops at the check of step 20 stays at level 21 while the
    other one goes on to an even level: each is read at its own parity."""
    quiet = dict(li.annulus(nr=40, nz=24, Ra=1e4, Da=1e-3), tol=10.0)
    other = li.annulus(nr=33, nz=50, Ra=1e5, Da=1e-3)
    lat = L.Lattice([quiet, other], storage=storage, check_interval=20)
    lat.step(40)
    assert lat.info(0)["status"] == "converged" and lat.info(0)["t"] == 21 and lat.info(1)["t"] == 40
    for i, (cfg, n) in enumerate(((quiet, 21), (other, 40))):
        one = L.Lattice([cfg], storage=storage, check_interval=0)
        one.step(n)
        same(lat.fields(i), one.fields(0), f"instance {i}")
        d = lat.fields_device(i)
        for k in ("uz", "ur", "p", "T"):
            np.testing.assert_array_equal(d[k].cpu().numpy(), one.fields(0)[k])
        one.close()
    lat.close()
