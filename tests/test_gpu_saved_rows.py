"""The saved buffers of a bfloat16 model step, given to gcn_layer_bwd: the
input rows lie where a layer call leaves them, also behind a layer whose
output width is not a multiple of 8."""
import numpy as np
import pytest
import torch

from gpu_util import require_gpu
from paper_1810_11899_amd import binding as B
from paper_1810_11899_amd import synth
from paper_1810_11899_amd.runner import StepRunner

pytestmark = pytest.mark.gpu


# widths of the first layer with 2h mod 8 in {2, 4, 6, 0}; vertex counts on
# both sides of the row-major weight gradient's least K (1024)
@pytest.mark.parametrize("order", [B.GCN_AGGREGATE_FIRST, B.GCN_TRANSFORM_FIRST])
@pytest.mark.parametrize("n", [700, 1500, 4099])
@pytest.mark.parametrize("h0", [33, 50, 75, 64])
def test_saved_of_a_step_serves_the_layer_call(h0, n, order):
    require_gpu()
    wl = synth.custom(n, "rmat", 9, [(50, h0), (2 * h0, 64)], head="ce", classes=13, seed=h0)
    r = StepRunner(wl, prec=B.GCN_BF16, orders=[order] * 2, first_layer_dH=True)
    dY = torch.randn((n, 128), generator=torch.Generator().manual_seed(n)).cuda()
    got = []
    for step in (r.step, r.step_calls):
        for t in r.saved:
            t.fill_(0xFF)      # NaN rows where nothing writes
        step()
        out = [torch.full_like(t, float("nan")) for t in (r.dH[1], r.dWs[1], r.dWn[1], r.db[1])]
        B.gcn_layer_bwd(r.A, r.AT, r.Y[0], r.W[1][0], r.W[1][1], r.Y[1], r.saved[1], dY, *out, order, r.ws, r.prec)
        got.append([t.cpu().numpy() for t in out])
    for x, y in zip(*got):
        assert np.isfinite(x).all() and np.array_equal(x.view(np.uint32), y.view(np.uint32))
