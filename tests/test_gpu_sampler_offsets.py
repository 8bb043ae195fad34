"""Induced subgraphs of a graph with 2^31 - 1 entries: rows whose last pieces
of 64 neighbours, and the rounds of eight loaded ahead, pass offset 2^31 - 1."""
import numpy as np
import pytest
import torch

from gpu_util import require_gpu
from paper_1810_11899_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("last", [1, 63, 64, 65, 512, 577, 600])
def test_rows_at_the_last_offsets(last):
    require_gpu()
    nnz = 2 ** 31 - 1
    lens = [577, 65, last]                       # rows 1, 2, 3; row 0 (not in the list) has the rest
    indptr = np.array([0, nnz - sum(lens), nnz - 65 - last, nnz - last, nnz], np.int32)
    rg = np.random.default_rng(last)
    tail = rg.integers(0, 4, sum(lens)).astype(np.int32)
    indices = torch.zeros(nnz, dtype=torch.int32, device="cuda")
    indices[-tail.size:] = torch.from_numpy(tail).cuda()
    G = B.DeviceCSR(4, 4, torch.from_numpy(indptr).cuda(), indices, torch.zeros(1, device="cuda"))
    lists = np.array([[3, 1, 2], [3, 3, 1]], np.int32)
    ib = B.InducedBatch(2, 3, 4096, "cuda")
    print(f"rows of {lens} at the end of 2^31 - 1 entries", flush=True)
    B.gcn_induce_subgraphs(G, torch.from_numpy(lists).cuda(), torch.tensor([3, 3], dtype=torch.int32).cuda(), ib,
                           B.Workspace())
    torch.cuda.synchronize()
    assert int(ib.status.item()) == 0
    off = ib.edge_offsets.cpu().numpy()
    for s, verts in enumerate(([1, 2, 3], [1, 3])):
        at = off[s]
        for i, v in enumerate(verts):
            r0 = int(indptr[v]) - (nnz - tail.size)
            row = tail[r0:r0 + lens[v - 1]]
            want = [verts.index(u) for u in row if u in verts]
            ip = ib.indptr[s].cpu().numpy()
            assert ip[i + 1] - ip[i] == len(want)
            assert np.array_equal(ib.indices[at + ip[i]:at + ip[i + 1]].cpu().numpy(), want)
    del indices, G
    torch.cuda.empty_cache()
