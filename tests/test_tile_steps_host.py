"""Several steps per launch on LDS tiles, checked on the host (no GPU).

A host build of the tile code (tests/tile_steps_host.hip) runs each tile as a
block of the kernel does and the same problem in single steps.  Every operation of
a node is the same on both paths, so the fields are bit-identical, in FP32 and
FP16 storage (whose stochastic rounding depends on the node's place), for every
side condition and for grids that the tiles cut evenly, raggedly or not at all.
No tile writes outside its buffer.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import lbm_inputs as li
from tests.test_wall_lanes_host import _init

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRC = os.path.join(HERE, "tile_steps_host.hip")
LIB = os.path.join(HERE, "libtile_steps_host.so")
DEPS = [SRC] + [os.path.join(ROOT, "paper_1409_5929_amd", "csrc", f)
                for f in ("lbm_axi_dev.h", "lbm_axi_desc.h", "lbm_axi_tile.h")]


def build_host_lib(force: bool = False) -> str:
    if force or not os.path.exists(LIB) or os.path.getmtime(LIB) < max(os.path.getmtime(f) for f in DEPS):
        hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
        subprocess.check_call([hipcc, "--offload-arch=gfx950", "-O2", "-std=c++17", "-shared", "-fPIC",
                               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                               "-I", os.path.join(ROOT, "include"), "-o", LIB + ".tmp", SRC])
        os.replace(LIB + ".tmp", LIB)
    return LIB


@pytest.fixture(scope="module")
def host():
    return ctypes.CDLL(build_host_lib())


CASES = {
    "annulus 66": (li.annulus(nr=66, nz=21, Ra=1e5, Da=1e-3), True),
    "annulus 65": (li.annulus(nr=65, nz=19, Ra=1e5, Da=1e-3), False),
    "three columns": (li.annulus(nr=3, nz=11, Ra=1e4, Da=1e-2), False),
    "nine columns": (li.annulus(nr=9, nz=4, Ra=1e4, Da=1e-2), False),
    "periodic ends": (dict(li.annulus(nr=30, nz=16, Ra=1e4, Da=1e-2), side_z="periodic", accel_z=1e-4), True),
    "pipe": (li.pipe(nr=40, nz=8), False),
    "heater": (li.heater_annulus(Da=1e-2, nr=40, nz=40), False),
    "inlet and outlet": (li.developing_pipe(Da=1e-2, nr=45, A=2.0, u_in=0.01), False),
    "cylinder": (dict(r0=0.5, side_rmin="axis", side_rmax="wall", side_z="wall", therm_rmin="adiabatic",
                      therm_rmax="fixed", therm_z="fixed", T_zmin=1.0, T_zmax=0.0, T_rmax=0.0, delta_T=1.0,
                      T_ref=0.5, L=20.0, phi=0.7, Da=1e-2, F_phi=-1.0, Ra=1e4, Pr=0.7, nr=21, nz=30), False),
}


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
@pytest.mark.parametrize("shape", [(2, 16, 5), (4, 16, 8), (4, 64, 7), (8, 32, 30), (10, 32, 12)], ids=str)
@pytest.mark.parametrize("name", CASES)
def test_tiles_equal_single_steps(host, name, shape, storage):
    from paper_1409_5929_amd import lbm

    cfg, field = CASES[name]
    m, vw, h = shape
    phi = np.ascontiguousarray(li.porosity_grf(cfg["nz"], cfg["nr"], seed=5), np.float32) if field else None
    init = np.ascontiguousarray(_init(cfg, 1409), np.float32)
    p = lbm.make_params(cfg, storage=storage, check_interval=0)
    ptr = lambda a: None if a is None else a.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    for wall_lanes in (0, 1):
        a, b = (np.zeros((4, cfg["nz"], cfg["nr"]), np.float32) for _ in range(2))
        rc = host.host_tile_steps(ctypes.byref(p), ptr(phi), ptr(init), 14, m, vw, h, wall_lanes, ptr(a), ptr(b))
        assert rc == 0, f"host_tile_steps returned {rc}"
        assert np.isfinite(b).all()
        np.testing.assert_array_equal(a, b, err_msg=f"{name}, wall lanes {wall_lanes}")


@pytest.mark.parametrize("nz", [8, 9, 11, 12, 40])
def test_periodic_rows_bound_the_steps_per_launch(host, nz):
    """A tile of a short periodic grid that takes more steps than the grid has
    rows would read rows that stand for none."""
    from paper_1409_5929_amd import lbm

    p = lbm.make_params(li.pipe(nr=40, nz=nz), storage="fp32", check_interval=0)
    most = ctypes.c_int()
    for m in range(2, 13, 2):
        inside = host.host_tile_inside(ctypes.byref(p), m, 32, 5, ctypes.byref(most))
        assert most.value == nz // 2 * 2
        assert inside == (1 if m <= nz else 0)
