"""The paired passes of small levels (residual with restriction, prolongation with a diagonal smoothing
step) at the edges of what they serve: level sizes around their workgroups, rows of A and of R of every
padded width, rows too long for them, FP64 and FP32, one and two smoothing steps. The sums keep their
order, so cycles are compared bit for bit with the separate passes (fusion off) and, in FP64, with the
oracle's within 1e-12."""
import numpy as np
import pytest
import scipy.sparse as sp

import workloads as W
from oracle import amg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def mesh(n, extra, seed):
    """Path graph of n nodes with `extra` random longer edges per node (row lengths vary with it)."""
    rng = np.random.default_rng(seed)
    i = np.concatenate([np.arange(n - 1), rng.integers(0, n, int(extra * n))])
    j = np.concatenate([np.arange(1, n), np.minimum(n - 1, np.concatenate([[0], i[n - 1:]])[1:] + rng.integers(1, 40, int(extra * n)))])
    keep = i != j
    i, j = np.minimum(i, j)[keep], np.maximum(i, j)[keep]
    key = np.unique(i * n + j)
    i, j = key // n, key % n
    w = rng.uniform(0.2, 1.0, i.size)
    L = sp.coo_matrix((np.concatenate([-w, -w]), (np.concatenate([i, j]), np.concatenate([j, i]))), shape=(n, n)).tocsr()
    L = (L + sp.diags(-np.asarray(L.sum(axis=1)).ravel() + 0.05)).tocsr()
    L.sort_indices()
    return W.CSRMatrix(L.indptr.astype(np.int32), L.indices.astype(np.int32), L.data.astype(np.float64), n, n)


@pytest.mark.parametrize("n,extra", [(33, 0.0), (64, 1.0), (257, 0.5), (1000, 2.0), (1023, 6.0), (2049, 12.0),
                                     (5000, 3.0), (16385, 1.0), (32768, 4.0), (32769, 1.0)])
def test_paired_cycles(n, extra):
    from paper_2606_19251_amd.solver import DeviceSolver, HostHierarchy

    A = mesh(n, extra, n)
    hier = HostHierarchy.build(A.rowptr, A.col, A.val, max_coarse=20)
    ds = DeviceSolver(hier)
    ds.set_jacobi()
    rng = np.random.default_rng(1)
    f, u0 = rng.standard_normal(n), rng.standard_normal(n)
    fd = torch.from_numpy(f).cuda()
    for precision in (64, 32):
        for nu1, nu2 in ((1, 1), (2, 2), (1, 0), (0, 1)):
            out = []
            for fused in (True, False):
                ds.set_fusion(fused)
                u = torch.from_numpy(u0.copy()).cuda()
                ds.vcycle(fd, u, nu1, nu2, precision)
                out.append(u.cpu().numpy())
            assert np.array_equal(out[0].view(np.uint64), out[1].view(np.uint64)), (n, precision, nu1, nu2)
    ds.set_fusion(True)
    xs = []
    for fused in (True, False):  # the outer loops' cycles start from a right-hand side with its first step
        ds.set_fusion(fused)
        xs.append(ds.solve(fd, precision=32, tol=1e-8)[0].cpu().numpy())
    assert np.array_equal(xs[0], xs[1])
    ho = amg.setup(amg.to_scipy(A), max_coarse=20)
    assert [l.A.shape[0] for l in ho.levels] == [L.n for L in hier.levels]
    ref = amg.vcycle(ho, amg.smoothers(ho, amg.jacobi_coeffs(2.0 / 3.0), 2), u0, f)
    ds.set_fusion(True)
    u = torch.from_numpy(u0.copy()).cuda()
    ds.vcycle(fd, u, 1, 1, 64)
    assert np.linalg.norm(u.cpu().numpy() - ref) <= 1e-12 * np.linalg.norm(ref)
    ds.close()
