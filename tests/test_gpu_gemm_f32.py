"""float32 products (split into bfloat16 parts on the matrix cores) against
float64, at tile edges and outside the split's range.

The products are reached through the layer calls on a graph without edges:
forward H W_self (NN), backward H^T dZ (TN) and dZ W_self^T (NT).
"""
import numpy as np
import pytest
import torch

from paper_1810_11899_amd import binding as B
from paper_1810_11899_amd import synth
from gpu_util import dev, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def run(H, Ws, dY):
    """(H Ws, H^T dY, dY Ws^T) through gcn_layer_fwd / gcn_layer_bwd."""
    n, f = H.shape
    h = Ws.shape[1]
    g = synth.empty_graph(n)
    A = B.DeviceCSR.from_host(n, n, g.indptr, g.indices, g.vals)
    ws = B.Workspace()
    order = B.GCN_TRANSFORM_FIRST
    Wn = torch.zeros((f, h), dtype=torch.float32, device="cuda")
    bias = torch.zeros(2 * h, dtype=torch.float32, device="cuda")
    Hd, Wd = dev(H), dev(Ws)
    out = []
    for sign in (1.0, -1.0):      # the two signs give the product behind the ReLU
        Y = torch.empty((n, 2 * h), dtype=torch.float32, device="cuda")
        B.gcn_layer_fwd(A, Hd, Wd * sign, Wn, bias, Y, None, order, ws)
        out.append(Y[:, :h].cpu().numpy())
    dYd = torch.zeros((n, 2 * h), dtype=torch.float32, device="cuda")
    dYd[:, :h] = dev(dY)
    Y = torch.ones((n, 2 * h), dtype=torch.float32, device="cuda")
    dH = torch.empty((n, f), dtype=torch.float32, device="cuda")
    dWs, dWn = (torch.empty((f, h), dtype=torch.float32, device="cuda") for _ in range(2))
    db = torch.empty(2 * h, dtype=torch.float32, device="cuda")
    B.gcn_layer_bwd(A, A, Hd, Wd, Wn, Y, None, dYd, dH, dWs, dWn, db, order, ws)
    return out[0], out[1], dWs.cpu().numpy(), dH.cpu().numpy()


def check(got, a, b, K, least=1e-37):
    """|got - a b| within three roundings per 16 k, the split's dropped parts
    and the split-K sums, each at most 2^-24 of sum |a||b|."""
    ref = a.astype(np.float64) @ b.astype(np.float64)
    mag = np.abs(a).astype(np.float64) @ np.abs(b).astype(np.float64)
    bound = (3.0 * K / 16 + 16 + 64) * 2.0 ** -24 * mag + least
    assert np.all(np.abs(got - ref) <= bound), float((np.abs(got - ref) / (mag + 1e-300)).max())


def norm_check(got, a, b):
    """The 2-norm error within 6e-7: three half-unit roundings per 16 k of sums
    that grow as a random walk, 2^-24 / sqrt(3) sqrt(3 k / 32), are 4.8e-7 for
    the 2050 k of a split of the longest sum here (the bound above, of the worst
    case, grows with K and would let products without their low parts pass;
    test_f32_split_host shows that this one does not)."""
    ref = a.astype(np.float64) @ b.astype(np.float64)
    assert np.linalg.norm(got - ref) <= 6e-7 * np.linalg.norm(ref)


# tile edges (64 / 128 / 256 rows, 64 / 128 columns, 16 k), remainders,
# unaligned widths, sizes on both sides of the rules for each tile, and splits
@pytest.mark.parametrize("n, f, h", [(1, 1, 1), (15, 17, 3), (127, 16, 129), (128, 128, 128), (129, 31, 127),
                                     (257, 33, 130), (300, 602, 41), (5000, 50, 64), (66000, 40, 260),
                                     (131072 + 77, 20, 20), (63, 65, 64), (64, 64, 63), (65, 63, 65), (8191, 256, 130),
                                     (16400, 300, 120), (1000, 1030, 190), (33000, 70, 65)])
def test_products_at_tile_edges(n, f, h):
    rg = np.random.default_rng(n + f + h)
    H = rg.standard_normal((n, f), dtype=np.float32) * np.exp2(rg.integers(-12, 12, (n, f))).astype(np.float32)
    Ws = rg.standard_normal((f, h), dtype=np.float32)
    dY = rg.standard_normal((n, h), dtype=np.float32) * 1e-4
    pos, neg, dW, dH = run(H, Ws, dY)
    for got, a, b, K in ((pos - neg, H, Ws, f), (dW, H.T, dY, n), (dH, dY, Ws.T, h)):
        check(got, a, b, K)
        norm_check(got, a, b)


@pytest.mark.parametrize("n, f, h", [(200, 48, 40), (66000, 48, 260)])
def test_products_outside_the_split_range(n, f, h):
    """Infinities, NaN, values above the largest bfloat16, overflowing sums
    and tiny operands give what float32 arithmetic gives."""
    rg = np.random.default_rng(n)
    H = rg.standard_normal((n, f), dtype=np.float32)
    Ws = rg.standard_normal((f, h), dtype=np.float32)
    Ws[:, 5] = np.abs(Ws[:, 5])
    H[3, 7] = np.inf
    H[4, 8] = -np.inf
    H[5, 9] = np.nan
    H[6] = 0.0
    H[6, 2] = np.float32(3.4e38)             # finite, rounds to infinity in bfloat16
    Ws[2, :20] = 0.25
    H[7, :] = np.float32(2e38)               # sums past float32's range
    H[8] *= np.float32(1e-36)
    H[9] *= np.float32(2.0 ** -100)
    dY = rg.standard_normal((n, h), dtype=np.float32)
    pos, neg, _, dH = run(H, Ws, dY)
    with np.errstate(all="ignore"):
        ref = H.astype(np.float64) @ Ws.astype(np.float64)
        ref32 = ref.astype(np.float32)
    rows = np.r_[0:3, 8:n]
    check(pos[rows] - neg[rows], H[rows], Ws, f)
    for r in (3, 4):
        assert np.all(np.isinf(pos[r]) == (ref32[r] > 0)) and np.all(np.isinf(neg[r]) == (ref32[r] < 0))
    # a NaN sum: what max(NaN, 0) leaves is never an infinity or a finite product
    assert not np.any(np.isinf(pos[5]) | (pos[5] > 0)) and not np.any(np.isinf(neg[5]) | (neg[5] > 0))
    assert np.allclose(pos[6, :20], 3.4e38 * 0.25, rtol=1e-6)
    assert np.isinf(pos[7, 5]) and neg[7, 5] == 0.0
    for r in (8, 9):
        mag = np.abs(H[r]).astype(np.float64) @ np.abs(Ws).astype(np.float64)
        assert np.all(np.abs(pos[r].astype(np.float64) - neg[r] - ref[r]) <= 1e-6 * mag + 1e-43)
    check(dH, dY, Ws.T, h)
    # the input gradient, without a ReLU behind it
    dY[0, 1], dY[1, 2] = np.inf, np.nan
    dY[2] = np.float32(1e-30)
    Ws2 = np.abs(Ws)
    _, _, _, dH = run(np.ones((n, f), np.float32), Ws2, dY)
    assert np.all(np.isposinf(dH[0])) and np.all(np.isnan(dH[1]))
    ref = dY[2].astype(np.float64) @ Ws2.T.astype(np.float64)
    assert np.allclose(dH[2], ref, rtol=2e-6, atol=0)


@pytest.mark.parametrize("n, f, h", [(200, 48, 40), (66000, 48, 260)])
@pytest.mark.parametrize("e", [-145, -135, -126, -118, -109, -60, 110])
def test_products_of_tiny_and_large(e, n, f, h):
    """Elements of about 2^e times elements of about 2^-e: ordinary sums of
    operands from the smallest subnormals up, to float32's own accuracy; and
    tiny elements beside ordinary ones that meet a zero."""
    rg = np.random.default_rng(n - e)
    tiny = lambda s: np.ldexp(rg.standard_normal(s), e).astype(np.float32)                       # noqa: E731
    large = lambda s: np.ldexp(rg.standard_normal(s), min(-e, 118) - 20).astype(np.float32)      # noqa: E731
    H, Ws = tiny((n, f)), large((f, h))
    H[::3, 5] = 1.0          # (the product's column 5 of H meets zeros)
    Ws[5] = 0.0
    dY = large((n, h))
    pos, neg, dW, _ = run(H, Ws, dY)
    check(pos - neg, H, Ws, f, 1e-43)
    rest = np.arange(f) != 5
    check(dW[rest], H[:, rest].T, dY, n, 1e-43)
    dY = tiny((n, h))
    _, _, dW, dH = run(large((n, f)), Ws, dY)
    check(dH, dY, Ws.T, h, 1e-43)


@pytest.mark.parametrize("K", [1, 2])
def test_shortest_sums(K):
    """One term is the rounded product; two are within two roundings of the
    larger magnitude (2 x 2^-24 of sum |a||b|)."""
    rg = np.random.default_rng(K)
    A, Bm = (rg.standard_normal(s, dtype=np.float32) for s in ((3000, K), (K, 160)))

    def shortest(got, a, b):
        ref = a.astype(np.float64) @ b.astype(np.float64)
        if K == 1:
            assert np.array_equal(got, ref.astype(np.float32))
        mag = np.abs(a).astype(np.float64) @ np.abs(b).astype(np.float64)
        assert np.all(np.abs(got - ref) <= 2.0 ** -23 * mag)

    pos, neg, _, _ = run(A, Bm, np.zeros((3000, 160), np.float32))
    shortest(pos - neg, A, Bm)
    _, _, dW, _ = run(np.ascontiguousarray(A.T), np.zeros((3000, 160), np.float32), Bm)     # n = K
    shortest(dW, A, Bm)
    if K == 1:    # the input gradient: K = 2h = 2, the other half's term zero
        _, _, _, dH = run(np.ones((3000, 160), np.float32), np.ascontiguousarray(Bm.T), A)
        shortest(dH, A, Bm)


# weight gradients on both sides of the 64 x 64 tiles' rules (2^30 multiply-adds,
# 16 tiles, one side in a tile) and of the 256-row tile's (no rows of padding)
@pytest.mark.parametrize("n, f, h", [(11000, 320, 140), (12000, 320, 150), (70000, 128, 128), (70000, 129, 128),
                                     (30000, 320, 64), (70000, 256, 300), (70000, 257, 300)])
def test_weight_gradients_at_the_tile_rules(n, f, h):
    rg = np.random.default_rng(n + f)
    H, dY = rg.standard_normal((n, f), dtype=np.float32), rg.standard_normal((n, h), dtype=np.float32)
    _, _, dW, _ = run(H, np.zeros((f, h), np.float32), dY)
    norm_check(dW, H.T, dY)
