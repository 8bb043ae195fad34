"""bfloat16 layers whose widths and vertex counts are not multiples of the
large-tile product's k-stage (32): padded input rows, K tails read as zeros,
narrow weight gradients; against the oracle, forward and backward."""
import numpy as np
import pytest
import torch

import test_gpu_layer as TL
from gpu_util import TOL_BF16, require_gpu
from paper_1810_11899_amd import binding as B
from paper_1810_11899_amd import synth

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


@pytest.mark.parametrize("f_in", [50, 203, 300, 602])     # padded to 56 (a column per lane), 208, 304, 608
def test_infinite_matrix_values_stay_infinite(f_in, ws):
    """An infinite value of A times the padding's zeros does not reach the
    outputs: with positive features and weights they are infinite."""
    n, h = 2000, 64
    g = synth.custom(n, "rmat", 9, [(f_in, h)], seed=f_in).graph
    deg = g.indptr[1:] - g.indptr[:-1]
    rows = np.array([int(deg.argmax()), int(np.flatnonzero(deg == 3)[0])])   # cut over wavefronts, and short
    vals = g.vals.copy()
    vals[g.indptr[rows]] = np.inf
    A = B.DeviceCSR.from_host(n, n, g.indptr, g.indices, vals)
    gen = torch.Generator().manual_seed(f_in)
    H, W = (torch.rand(s, generator=gen).add_(0.5).cuda() for s in ((n, f_in), (f_in, h)))
    Y = torch.empty((n, 2 * h), device="cuda")
    order = B.GCN_AGGREGATE_FIRST
    saved = torch.empty(B.gcn_layer_saved_bytes(n, f_in, h, order, B.GCN_BF16), dtype=torch.uint8, device="cuda")
    B.gcn_layer_fwd(A, H, W, W, torch.zeros(2 * h, device="cuda"), Y, saved, order, ws, B.GCN_BF16)
    neigh = Y[:, h:].cpu().numpy()
    assert np.isposinf(neigh[rows]).all() and np.isfinite(np.delete(neigh, rows, 0)).all()


# both sides of the large tile's rules for forward and input-gradient products:
# one head launch of 127 / 129 blocks of 256 rows, 32 / 33 classes; two products
# a launch of 126 / 130 blocks; 78 / 80 blocks of wide ones; rows of N mod 4
@pytest.mark.parametrize("n, f, C", [(32512, 64, 33), (33024, 64, 32), (33024, 64, 33), (33000, 64, 41)])
def test_head_at_the_large_tile_rules(n, f, C, ws):
    TL.test_loss_grad(B.GCN_BF16, TOL_BF16, "ce", n, f, C, ws)


@pytest.mark.parametrize("shape", [(16128, "er", 4, 72, 40), (16640, "er", 4, 72, 40), (9984, "er", 4, 56, 136),
                                   (10240, "er", 4, 56, 136), (20500, "er", 4, 130, 8), (20500, "er", 4, 134, 104)])
def test_layer_at_the_large_tile_rules(shape, ws):
    TL.test_layer_forward(B.GCN_BF16, TOL_BF16, B.GCN_AGGREGATE_FIRST, shape, ws)
    TL.test_layer_backward(B.GCN_BF16, TOL_BF16, B.GCN_AGGREGATE_FIRST, True, shape, ws)


# operands read element by element on both sides of the 64 x 64 tiles' rule:
# weight gradients of 4.4, 4.8 and (one tile wide) 6.2e8 multiply-adds in whole
# tiles, forward and input-gradient products of 7.8 and 8.3e8
@pytest.mark.parametrize("shape", [(4203, "er", 4, 202, 201), (4603, "er", 4, 202, 201), (15001, "er", 4, 301, 61),
                                   (1985, "er", 4, 602, 301), (2115, "er", 4, 602, 301)])
def test_elementwise_operands_at_the_tile_rule(shape, ws):
    TL.test_layer_forward(B.GCN_BF16, TOL_BF16, B.GCN_AGGREGATE_FIRST, shape, ws)
    TL.test_layer_backward(B.GCN_BF16, TOL_BF16, B.GCN_TRANSFORM_FIRST, True, shape, ws)
