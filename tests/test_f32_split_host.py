"""The float32 products' three-part bfloat16 split, modelled in numpy: exact
over float32's whole range, and what the GPU tests' 2-norm bound can tell."""
import numpy as np
import pytest

SCALE = 24                 # elements times 2^24 before the split
BOUND = 6e-7               # test_gpu_gemm_f32.norm_check


def bf16(x):
    u = x.astype(np.float32).view(np.uint32).astype(np.uint64)
    r = (u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000
    return r.astype(np.uint32).view(np.float32)


def split(x, scale=SCALE):
    x = np.ldexp(x, scale).astype(np.float32)
    h = bf16(x)
    m = bf16(x - h)
    return h, m, bf16(x - h - m)


@pytest.mark.parametrize("e", [-149, -140, -133, -127, -126, -118, -109, -90, 0, 60, 102])
def test_split_is_exact_and_normal(e):
    """h + m + l is the scaled element and no part is a subnormal; without the
    scaling the parts lose bits below 2^-110."""
    rg = np.random.default_rng(e + 200)
    x = np.ldexp(rg.integers(2 ** 23, 2 ** 24, 4096).astype(np.float64) * rg.choice([-1, 1], 4096), e - 23)
    x = x.astype(np.float32)                 # (below 2^-126 rounded to subnormals)
    parts = split(x)
    total = sum(p.astype(np.float64) for p in parts)
    assert np.array_equal(total, np.ldexp(x.astype(np.float64), SCALE))
    nz = np.concatenate([np.abs(p[p != 0]) for p in parts])
    assert nz.size == 0 or nz.min() >= 2.0 ** -126
    unscaled = sum(p.astype(np.float64) for p in split(x, 0))
    assert np.array_equal(unscaled, x.astype(np.float64)) == (e >= -110)


@pytest.mark.parametrize("K", [64, 1024, 131072])
def test_bound_tells_missing_parts(K):
    """Products without m m', h l' and l h', or of the leading parts alone,
    exceed the bound at every K; all six part products stay below it."""
    rg = np.random.default_rng(K)
    A = rg.standard_normal((20, K), dtype=np.float32) * np.exp2(rg.integers(-12, 12, (20, K))).astype(np.float32)
    Bm = rg.standard_normal((K, 20), dtype=np.float32)
    ref = A.astype(np.float64) @ Bm.astype(np.float64)
    a, b = ([p.astype(np.float64) for p in split(x)] for x in (A, Bm))
    err = lambda pairs: np.linalg.norm(np.ldexp(sum(a[i] @ b[j] for i, j in pairs), -2 * SCALE) - ref) / np.linalg.norm(ref)  # noqa: E731
    assert err([(0, 0)]) > 100 * BOUND
    assert err([(0, 0), (0, 1), (1, 0)]) > 3 * BOUND
    assert err([(0, 0), (0, 1), (1, 0), (1, 1)]) > 3 * BOUND          # no l parts
    assert err([(0, 0), (0, 1), (1, 0), (1, 1), (0, 2), (2, 0)]) < 0.1 * BOUND
