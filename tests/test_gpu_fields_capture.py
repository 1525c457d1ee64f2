"""Field reads on a stream that is being captured are refused, at every size.

What a field read launches follows the parity of the time level at the call (the AA
layout), so a graph that recorded it would read the wrong slots when replayed at
the other parity.  The refusal leaves the capture and the handle as they were.
"""
import ctypes

import pytest

import lbm_inputs as li
from tests.test_gpu_batch import L, same  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("check", [0, 50])
@pytest.mark.parametrize("nr,nz", [(64, 48), (512, 4200)])  # the second above 8192 tiles
def test_field_reads_are_refused_during_capture(L, nr, nz, check):  # noqa: F811
    import torch

    s = torch.cuda.Stream()
    lat = L.Lattice(li.pipe(nr=nr, nz=nz), check_interval=check, stream=s.cuda_stream)
    lat.step(12)
    lat.sync()
    before = lat.fields(0)
    out = torch.zeros((nz, nr), dtype=torch.float32, device="cuda")
    mx = torch.zeros(1, dtype=torch.float64, device="cuda")
    other = torch.zeros(4, device="cuda")
    torch.cuda.synchronize()
    lib, h, p = lat._lib, lat._h, ctypes.c_void_p(out.data_ptr())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        graph.capture_begin(capture_error_mode="thread_local")
        other.add_(1.0)
        got = [lib.lbm_axi_macros(h, 0, p, None, None, None, None, 1),
               lib.lbm_axi_density_deviation(h, 0, p, 1),
               lib.lbm_axi_stream_function_static(h, 0, p, ctypes.c_void_p(mx.data_ptr()))]
        graph.capture_end()
    assert got == [-3, -3, -3], got  # LBM_AXI_EDEVICE
    graph.replay()
    torch.cuda.synchronize()
    assert other.tolist() == [1.0] * 4 and out.abs().max().item() == 0.0
    same(lat.fields(0), before, "after the capture")
    lat.step(5)
    assert lat.info()["t"] == 17
    lat.close()
