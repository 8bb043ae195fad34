"""bfloat16 layers whose widths and vertex counts are not multiples of the
large-tile product's k-stage (32): padded input rows, K tails read as zeros,
narrow weight gradients; against the oracle, forward and backward."""
import pytest
import torch

import test_gpu_layer as TL
from gpu_util import TOL_BF16, require_gpu
from paper_1810_11899_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ws():
    require_gpu()
    yield B.Workspace("cuda")
    torch.cuda.synchronize()


# (n, graph, d, f_in, h): n mod 32 in {1, 3, 7, 31, 0}, f_in mod 8 and mod 32
# over their range, h a multiple of 8 (large tile) and not (the other kernel),
# sides on both sides of the large tile's rules (32, 128; K of 1024)
SHAPES = [(1025, "rmat", 9, 602, 64), (4099, "rmat", 9, 50, 64), (2047, "er", 8, 371, 40), (1031, "rmat", 9, 200, 264),
          (3001, "er", 7, 33, 32), (8003, "rmat", 9, 130, 128), (777, "rmat", 9, 300, 136), (1056, "er", 9, 8, 256),
          (1024, "rmat", 8, 257, 36), (1023, "rmat", 8, 72, 24), (5000, "rmat", 9, 31, 24)]


@pytest.mark.parametrize("order", [B.GCN_AGGREGATE_FIRST, B.GCN_TRANSFORM_FIRST])
@pytest.mark.parametrize("shape", SHAPES)
def test_ragged_layer(order, shape, ws):
    print(f"bf16 ragged layer {shape} order {order}", flush=True)
    TL.test_layer_forward(B.GCN_BF16, TOL_BF16, order, shape, ws)
    for want_dH in (True, False):
        TL.test_layer_backward(B.GCN_BF16, TOL_BF16, order, want_dH, shape, ws)


@pytest.mark.parametrize("kind", ["ce", "bce"])
@pytest.mark.parametrize("n, f, C", [(1025, 264, 41), (4099, 128, 100), (1033, 68, 33), (2047, 1000, 31), (16385, 72, 5)])
def test_ragged_head(kind, n, f, C, ws):
    TL.test_loss_grad(B.GCN_BF16, TOL_BF16, kind, n, f, C, ws)
