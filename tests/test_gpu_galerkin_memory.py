"""What amgg_galerkin_device holds while it compacts its result: the intermediate product A P and R = P^T are
released before, in the row-wise and in the expanding form, and the expanding form starts without the
row-wise form's temporaries."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import amg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev(M):
    return tuple(torch.from_numpy(a).cuda() for a in (M.indptr.astype(np.int32), M.indices.astype(np.int32), M.data))


def problem(hub):
    """A path graph of pairs (P sums pairs) with every fourth coupling between the pairs cancelling exactly, so
    that zeros are dropped; optionally a hub row of more products than the row-wise form serves."""
    n = 20000
    rows = np.arange(n)
    upper = np.where(np.arange(n - 1) % 4 == 1, 0.5, -1.0)
    d = sp.diags([upper, np.full(n, 4.0), np.full(n - 1, -1.0)], [1, 0, -1]).tolil()
    for i in range(1, n - 3, 4):  # the block between pair (i - 1, i) and the next: 0.5 - 0.5
        d[i - 1, i + 1] = -0.5
    A = d.tocsr()
    if hub:
        c = np.arange(5, n, 2)
        A = (A + sp.csr_matrix((np.full(c.size, -0.25), (np.full(c.size, 3), c)), shape=A.shape)).tocsr()
    A.sort_indices()
    P = sp.csr_matrix((np.ones(n), (rows, rows // 2)), shape=(n, n // 2))
    return A, P


@pytest.mark.parametrize("hub", [False, True])
@pytest.mark.parametrize("chunk", [0, 100000])
def test_operands_are_released_before_the_compaction(hub, chunk):
    from paper_2606_19251_amd import capi

    class Log(capi.TorchDeviceAllocator):
        """Sizes held whenever something is allocated."""

        def __init__(self):
            super().__init__(torch, torch.device("cuda", 0))
            self.held = []

        def _alloc(self, nbytes, user):
            self.held.append([t.numel() for t in self.live.values()])
            return super()._alloc(nbytes, user)

    A, P = problem(hub)
    AP = amg.spgemm_rowwise_vec(A, P)
    ref = amg.galerkin(A, P)
    full = amg.spgemm_rowwise_vec(amg.transpose_exact(P), AP).nnz
    assert ref.nnz < full  # something is dropped
    al = Log()
    got = capi.amgg_galerkin_device(0, A.shape[0], P.shape[1], *dev(A), *dev(P), chunk_products=chunk, allocator=al)
    for g, r in zip(got, (ref.indptr, ref.indices, ref.data)):
        assert np.array_equal(g.cpu().numpy(), r)
    at_end = al.held[-1]  # before the last array of the result
    ap, r_val = 8 * AP.nnz, 8 * P.nnz
    assert ap not in (8 * ref.nnz, 8 * full, r_val) and ap not in at_end and r_val not in at_end
    if hub and chunk == 0:  # the first product is expanded: nothing of the row-wise attempt is held by then
        # the flags, R's three arrays, the transpose's cursor, the product's row pointer, the rows of A's entries
        expanding = next(h for h in al.held if 4 * A.nnz in h)
        assert len(expanding) == 7
