"""The network's GEMM block shapes on the GPU: which one a layer takes follows its
rows and pixels, and every shape adds the products of an output in the same
order, so a sample's result does not depend on the batch it is in, bit for bit.
Batch 1 runs on the smallest blocks, the largest batches on the largest (those
are held to the FP64 oracle in test_gpu_no.py); gradients, whose sums over the
pixels are split by batch, are held to the oracle here, with its tolerance
(bfloat16 operands, FP32 sums over 8 layers: 3e-2)."""
import numpy as np
import pytest

import lbm_inputs as li
from oracle import no_oracle as N
from tests.test_gpu_no import TOL, rel, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def draw(widths, H, W, B, seed):
    rng = np.random.default_rng(seed)
    params = li.no_init_params(widths, seed=seed)
    params = params + (0.05 * rng.standard_normal(params.size)).astype(np.float32)
    return params, rng.standard_normal((B, 6, H, W)).astype(np.float32), rng.standard_normal((B, 3, H, W)).astype(np.float32)


@pytest.mark.parametrize("widths,H,W,batches", [
    ((48, 96, 192, 384), 128, 128, (32, 8, 3, 1)),  # 48 and 96 rows: blocks without padding
    ((32, 64, 128, 256), 128, 64, (64, 16, 1)),
    ((34, 66, 98, 130), 64, 72, (40, 7, 1)),  # ragged rows and pixels
    ((2, 2, 2, 2), 8, 8, (64, 1)),
    ((8, 16, 24, 32), 8, 40, (33, 2, 1)),  # pixel counts that are no multiple of 8
])
def test_a_sample_does_not_depend_on_its_batch(torch, widths, H, W, batches):  # noqa: F811
    from paper_1409_5929_amd.no import WarmStartNet

    params, x, _ = draw(widths, H, W, batches[0], 31)
    xs = torch.from_numpy(x).cuda()
    net = WarmStartNet(widths, H, W, batches[0], params)
    ref = net.forward(xs).cpu().numpy()
    assert np.isfinite(ref).all()
    for b in batches[1:]:
        for at in (0, batches[0] - b):
            y = net.forward(xs[at:at + b].contiguous()).cpu().numpy()
            np.testing.assert_array_equal(y, ref[at:at + b])
    net.close()


@pytest.mark.parametrize("widths,H,W,B", [((34, 66, 98, 130), 24, 40, 1), ((48, 96, 192, 384), 32, 32, 1),
                                          ((8, 16, 24, 32), 8, 8, 1)])
def test_small_problems_match_oracle(torch, widths, H, W, B):  # noqa: F811
    from paper_1409_5929_amd.no import WarmStartNet

    params, x, t = draw(widths, H, W, B, 32)
    net = WarmStartNet(widths, H, W, B, params)
    y = net.forward(torch.from_numpy(x).cuda()).cpu().numpy()
    loss = net.gradients(torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda())
    g = net.grads()
    net.close()
    p64 = params.astype(np.float64)
    ref, _ = N.forward(p64, widths, x.astype(np.float64))
    lref, gref = N.loss_and_grads(p64, widths, x.astype(np.float64), t.astype(np.float64))
    assert rel(y, ref) <= TOL and rel(g, gref) <= TOL and abs(loss - lref) <= TOL * lref
