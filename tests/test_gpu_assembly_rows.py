"""Smoother assembly (Eq. 5) at the edges of its row blocks: the rows per workgroup follow from the
row count and the mean row length, so banded matrices of several widths and of sizes around every
block size are compared, bit for bit, with the oracle's values (each operation is rounded on its own
on both sides, so the tolerance is zero)."""
import numpy as np
import pytest
import scipy.sparse as sp

import workloads as W
from oracle import amg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def banded(n, w, seed):
    rng = np.random.default_rng(seed)
    i = np.concatenate([np.arange(n - k) for k in range(1, w + 1)])
    j = np.concatenate([np.arange(k, n) for k in range(1, w + 1)])
    v = rng.uniform(0.5, 2.0, i.size) * np.where(rng.uniform(size=i.size) < 0.1, 1e-3, 1.0)
    L = sp.coo_matrix((np.concatenate([-v, -v]), (np.concatenate([i, j]), np.concatenate([j, i]))), shape=(n, n)).tocsr()
    L = (L + sp.diags(-np.asarray(L.sum(axis=1)).ravel() + 0.1)).tocsr()
    L.sort_indices()
    return W.CSRMatrix(L.indptr.astype(np.int32), L.indices.astype(np.int32), L.data.astype(np.float64), n, n)


@pytest.mark.parametrize("n,w", [(1, 0), (15, 3), (16, 3), (17, 5), (33, 30), (497, 60), (8191, 2), (8193, 30),
                                 (16385, 12), (33000, 5), (65537, 3), (131073, 2)])
def test_assembly_bitwise(n, w):
    from paper_2606_19251_amd.solver import DeviceSolver, HostHierarchy

    A = banded(n, w, n) if w else W.CSRMatrix(np.array([0, 1], np.int32), np.zeros(1, np.int32), np.ones(1), 1, 1)
    ds = DeviceSolver(HostHierarchy.build(A.rowptr, A.col, A.val))
    c = np.array([0.62, 0.031, -0.004, 0.21, 0.017])
    ds.set_coeffs_device(torch.from_numpy(np.tile(c.astype(np.float32), (ds.nlevels, 1))).cuda(), 2)
    torch.cuda.synchronize()
    for l, L in enumerate(ds.hier.levels):
        if L.nnz == L.n:
            continue  # a diagonal matrix has no off-diagonal scale
        S = sp.csr_matrix((L.val, L.col, L.rowptr), shape=(L.n, L.n))
        ref = amg.assemble_smoother(S, c.astype(np.float32).astype(np.float64), 2)
        v = ds.level_view(l)
        got = v["q_val"].cpu().numpy()
        assert np.array_equal(got.view(np.uint64), np.ascontiguousarray(ref.data).view(np.uint64)), (n, w, l)
        assert np.array_equal(v["q_val32"].cpu().numpy(), ref.data.astype(np.float32))
    ds.close()
