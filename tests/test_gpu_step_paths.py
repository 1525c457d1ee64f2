"""Which way plain steps are launched, and that every way gives the same bits.

lbm_axi_step takes plain steps several to a launch on LDS tiles, in replays of a
captured graph, or one by one.  step_paths() counts the steps of each, so that a
comparison of two ways is known to be one.
"""
import numpy as np
import pytest

import lbm_inputs as li
from tests.test_gpu_batch import L, same  # noqa: F401
from tests.test_gpu_tile_steps import CASES
from tests.test_wall_lanes_host import _init

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("name", CASES)
def test_long_runs_take_tiles_and_short_or_timed_ones_do_not(L, name, storage):  # noqa: F811
    cfgs, field = CASES[name]
    phi = [li.porosity_grf(c["nz"], c["nr"], seed=3) for c in cfgs] if field else None
    lat = L.Lattice(cfgs, phi=phi, storage=storage, check_interval=50)
    assert lat.step_paths() == {"single": 0, "graph": 0, "tiles": 0}
    lat.step(61)  # the check steps 0 and 50 and the odd level after each, then 48 and 8 plain steps
    assert lat.step_paths() == {"single": 5, "graph": 0, "tiles": 56}
    for _ in range(4):
        lat.step(3)
    lat.set_timing(True)
    lat.step(20)
    assert lat.step_paths() == {"single": 37, "graph": 0, "tiles": 56}
    lat.close()


def test_no_graphs_means_single_launches_and_no_second_planes(L):  # noqa: F811
    """set_graph(0) gives the memory of the second set of planes back, any other value takes it again."""
    cfg = li.annulus(nr=96, nz=72, Ra=1e5, Da=1e-3)
    lat, other = (L.Lattice(cfg, check_interval=0) for _ in range(2))
    planes = 14 * 128 * 72 * 4  # rows are padded to 64 columns
    both = lat.info()["device_bytes"]
    lat.set_graph(0)
    assert planes <= both - lat.info()["device_bytes"] <= planes + 4096
    lat.step(40)
    assert lat.step_paths() == {"single": 40, "graph": 0, "tiles": 0}
    lat.set_storage("fp32")  # does not bring it back
    lat.step(2)
    lat.set_wall_lanes(0)
    lat.set_wall_lanes(-1)
    lat.step(8)
    assert lat.step_paths()["tiles"] == 0 and both - lat.info()["device_bytes"] >= planes
    lat.set_graph(8)
    assert lat.info()["device_bytes"] == both
    lat.step(50)
    assert lat.step_paths() == {"single": 50, "graph": 0, "tiles": 50}
    other.step(100)
    same(lat.fields(0), other.fields(0), "single launches, then tiles")
    lat.close()
    other.close()


@pytest.mark.parametrize("change", ["storage", "wall lanes"])
def test_a_step_allocates_nothing(L, change):  # noqa: F811
    """What the second set of planes rests on may change under a handle: the call that
    changes it takes the new set, not the next step."""
    lat = L.Lattice(li.annulus(nr=96, nz=72, Ra=1e5, Da=1e-3), storage="fp16", check_interval=0)
    lat.step(20)
    if change == "storage":
        lat.set_storage("fp32")
    else:
        lat.set_wall_lanes(0)
    held = lat.info()["device_bytes"]
    lat.step(20)
    assert lat.step_paths()["tiles"] == 40 and lat.info()["device_bytes"] == held
    lat.close()


def test_second_planes_of_all_handles_are_bounded(L):  # noqa: F811
    """Handles that each take a fiftieth of the device's memory: three have second sets of
    planes (a sixteenth in all), the next ones single steps with the same bits, until one is
    closed."""
    import torch

    total = torch.cuda.mem_get_info()[1]
    nz = total // 50 // (14 * 4 * 8192)
    cfg = li.annulus(nr=8192, nz=int(nz), Ra=1e5, Da=1e-3)
    planes = 14 * 4 * 8192 * int(nz)
    held = lambda lat: lat.info()["device_bytes"] // planes  # noqa: E731
    lats = [L.Lattice(cfg, check_interval=0) for _ in range(5)]
    assert [held(lat) for lat in lats] == [2, 2, 2, 1, 1]
    for lat in (lats[0], lats[4]):
        lat.step(8)
    a, b = lats[0].fields_device(0), lats[4].fields_device(0)
    assert lats[0].step_paths()["tiles"] == 8 and lats[4].step_paths()["tiles"] == 0
    assert all(torch.equal(a[k], b[k]) for k in a)
    lats.pop(1).close()
    lats.append(L.Lattice(cfg, check_interval=0))
    assert [held(lat) for lat in lats] == [2, 2, 1, 1, 2]
    for lat in lats:
        lat.close()


def _periodic(nr, nz):
    return dict(li.annulus(nr=nr, nz=nz, Ra=1e4, Da=1e-2), r0=200.0, side_rmin="periodic", side_rmax="periodic",
                side_z="periodic", accel_z=1e-5)


GRAPHS = {  # problems whose plain steps are not taken on tiles
    "radially periodic": ([_periodic(70, 24)], ("fp32", "fp16")),
    "two radially periodic": ([_periodic(70, 24), _periodic(40, 33)], ("fp32", "bf16")),
    "a 16-bit grid of more than one round of tiles": ([li.annulus(nr=760, nz=690, Ra=1e5, Da=1e-3)], ("fp16", "bf16")),
}


@pytest.mark.parametrize("G", [8, 32])
@pytest.mark.parametrize("name,storage", [(n, s) for n in GRAPHS for s in GRAPHS[n][1]])
def test_graph_replays_equal_single_steps(L, name, storage, G):  # noqa: F811
    """Replays with check steps, field reads and synchronisations between them, and
    odd starts: each against a handle without graphs."""
    cfgs = GRAPHS[name][0]
    init = [_init(c, 7) for c in cfgs]
    for a in init:
        a[:2] *= 0.1
    graph, single = (L.Lattice(cfgs, init=init, storage=storage, check_interval=100) for _ in range(2))
    graph.set_graph(G)
    single.set_graph(0)
    for n in (1, 37, 64, 3, 45):
        graph.step(n)
        single.step(n)
        for i in range(len(cfgs)):
            f = graph.fields(i)
            assert all(np.isfinite(f[k]).all() for k in ("uz", "ur", "T"))
            same(f, single.fields(i), f"{name} {storage} G={G} instance {i}, {graph.info()['t']} steps")
    a, b = graph.residual(), single.residual()
    for k in ("res", "nu_i", "nu_o", "status"):
        np.testing.assert_array_equal(a[k], b[k])
    # from the first even level on, as many replays as fit before the end of a call or the check step
    replayed = sum(n // G * G for n in (36, 62, 2, 44))
    assert graph.step_paths() == {"single": 150 - replayed, "graph": replayed, "tiles": 0}
    assert single.step_paths() == {"single": 150, "graph": 0, "tiles": 0}
    graph.close()
    single.close()
