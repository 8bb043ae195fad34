"""Transposition and validation of a matrix with 2^31 - 1 entries, whose last
rows are walked 16, 64 and 512 entries at a time up to the last offset."""
import numpy as np
import pytest
import torch

from gpu_util import require_gpu
from paper_1810_11899_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("last", [1, 40, 65, 577])
def test_rows_at_the_last_offsets(last):
    require_gpu()
    nnz, lens, N = 2 ** 31 - 1, [577, 65, last], 2 ** 20
    tail = sum(lens)                   # entries of the rows N, N + 1, N + 2; the others hold column 0 only
    indptr = np.r_[np.linspace(0, nnz - tail, N + 1).astype(np.int64), nnz - tail + np.cumsum(lens)]
    rg = np.random.default_rng(last)
    choice = rg.integers(0, 4, tail)
    cols, vals = np.array([0, N, N + 1, N + 2], np.int32)[choice], rg.standard_normal(tail).astype(np.float32)
    ix = torch.zeros(nnz, dtype=torch.int32, device="cuda")
    vv = torch.ones(nnz, dtype=torch.float32, device="cuda")
    ix[-tail:], vv[-tail:] = torch.from_numpy(cols).cuda(), torch.from_numpy(vals).cuda()
    A = B.DeviceCSR(N + 3, N + 3, torch.from_numpy(indptr.astype(np.int32)).cuda(), ix, vv)
    print(f"rows of {lens} at the end of 2^31 - 1 entries: general transposition", flush=True)
    AT = B.gcn_csr_transpose(A, B.Workspace())
    rows = np.repeat([N, N + 1, N + 2], lens)
    k = int((cols > 0).sum())
    order = np.argsort(choice[cols > 0], kind="stable")
    first = nnz - k + np.cumsum(np.r_[0, np.bincount(choice, minlength=4)[1:]])
    got = AT.indptr.cpu().numpy()
    assert got[0] == 0 and (got[1:N + 1] == nnz - k).all() and np.array_equal(got[N:], first)
    assert np.array_equal(AT.indices[-k:].cpu().numpy(), rows[cols > 0][order])
    assert np.array_equal(AT.vals[-k:].cpu().numpy(), vals[cols > 0][order])
    del AT
    torch.cuda.empty_cache()
    print("validation", flush=True)
    assert B.gcn_csr_validate(A, require_sorted=False).cpu().tolist() == [0, 0]
    ix[-1] = N + 3
    assert B.gcn_csr_validate(A, require_sorted=False).cpu().tolist() == [3, N + 2]
    print("values of the symmetric transposition, rows of one value each", flush=True)
    ix[-1], choice[-1] = N + 2, 3
    vv[-tail:] = torch.from_numpy((rows - N + 2).astype(np.float32)).cuda()
    t = B.gcn_csr_transpose_symmetric(A, B.Workspace()).vals
    assert np.array_equal(t[-tail:].cpu().numpy(), np.array([1, 2, 3, 4], np.float32)[choice])
    assert bool((t[:nnz - tail] == 1).all())
    del A, ix, vv, t
    torch.cuda.empty_cache()
