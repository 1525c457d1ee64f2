"""Which cuts of a grid into LDS tiles are taken (no GPU).

A tile whose region ended beside a radial wall column that it leaves out gave other
random bits to the boundary nodes next to that column: in 16-bit storage with
wall lanes its nodes were not those of single steps.  Such cuts are refused; the
cuts that the library makes (32 columns, up to 8 steps) are all taken, and any cut
that is taken gives the bits of single steps.
"""
import ctypes

import numpy as np
import pytest

import lbm_inputs as li
from tests.test_tile_steps_host import host  # noqa: F401
from tests.test_wall_lanes_host import _init


def _inside(host, cfg, m, vw, h):  # noqa: F811
    from paper_1409_5929_amd import lbm

    p = lbm.make_params(cfg, storage="fp16", check_interval=0)
    return host.host_tile_inside(ctypes.byref(p), m, vw, h, ctypes.byref(ctypes.c_int()))


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
@pytest.mark.parametrize("nr", range(9, 20))
def test_cuts_taken_equal_single_steps(host, nr, storage):  # noqa: F811
    from paper_1409_5929_amd import lbm

    cfg = li.annulus(nr=nr, nz=14, Ra=1e5, Da=1e-2)
    p = lbm.make_params(cfg, storage=storage, check_interval=0)
    init = np.ascontiguousarray(_init(cfg, 3), np.float32)
    ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    for m, vw in ((2, 6), (4, 10), (6, 14)):
        taken = _inside(host, cfg, m, vw, 5)
        for wall_lanes in (0, 1):
            a, b = (np.zeros((4, cfg["nz"], nr), np.float32) for _ in range(2))
            rc = host.host_tile_steps(ctypes.byref(p), None, ptr(init), 12, m, vw, 5, wall_lanes, ptr(a), ptr(b))
            assert rc == (0 if taken else -2)
            if taken:
                np.testing.assert_array_equal(a, b, err_msg=f"{m} steps, {vw} columns, wall lanes {wall_lanes}")


def test_a_region_beside_a_wall_it_leaves_out_is_refused(host):  # noqa: F811
    assert _inside(host, li.annulus(nr=11, nz=14, Ra=1e5, Da=1e-2), 4, 10, 5) == 0  # cut at column 5: region from 1


@pytest.mark.parametrize("cfg", [li.annulus(nr=65, nz=19, Ra=1e5, Da=1e-3), li.pipe(nr=40, nz=12)], ids=["annulus", "pipe"])
def test_every_cut_the_library_makes_is_taken(host, cfg):  # noqa: F811
    for nr in list(range(4, 200)) + [641, 1025, 4096, 8192]:
        for m in (2, 4, 6, 8):
            assert _inside(host, dict(cfg, nr=nr), m, 32, 28) == 1, (nr, m)
