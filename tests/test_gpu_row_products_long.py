"""Row-wise Galerkin products at both sides of every limit between the kernels that serve a row, the product
counts taken from the matrices: full tables and full sorts (as many different columns as products), many
products per column, rows of the prolongation without entries, and one row beyond the longest, which sends
the product to the expanding form. Against the oracle's products bit for bit (the accumulation order is
the same)."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import amg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LIMITS = (32, 128, 1024, 2048, 8192)  # most products of a row, by class


def dev(M):
    return tuple(torch.from_numpy(a).cuda() for a in (M.indptr.astype(np.int32), M.indices.astype(np.int32), M.data))


def csr(rows, cols, shape, rng):
    M = sp.csr_matrix((rng.uniform(-1.0, 1.0, len(rows)), (rows, cols)), shape=shape)
    M.sort_indices()
    return M


def products(L, M):
    """Products of every row of L M."""
    return np.add.reduceat(np.append(np.diff(M.indptr)[L.indices], 0), L.indptr[:-1]) * (np.diff(L.indptr) > 0)


def problem(kind, longest):
    """A with a row of every limit and one more (up to `longest` products) among short rows, and P."""
    rng = np.random.default_rng(5)
    n = 9000
    want = sorted({c for m in LIMITS for c in (m - 1, m, m + 1)} - {8191, 8192, 8193} | {longest - 1, longest})
    if kind == "distinct":  # P the identity: every product has a column of its own
        nc, length = n, np.ones(n, int)
        P = csr(np.arange(n), np.arange(n), (n, n), rng)
    else:  # rows of 0, 1 and 2 entries in 1500 columns; the columns of the long rows' points are theirs alone
        nc = 1500
        length = rng.integers(0, 3, n)
        long_rows = 7 + 300 * np.arange(len(want))
        length[long_rows] = 1
        c = [np.sort(rng.choice(nc - len(want), k, replace=False)) for k in length]
        for k, i in enumerate(long_rows):
            c[i] = np.array([nc - len(want) + k])
        P = csr(np.repeat(np.arange(n), length), np.concatenate(c), (n, nc), rng)
    rows, cols = [], []
    two, one = np.flatnonzero(length == 2), np.flatnonzero(length == 1)
    for i in range(n):
        k, off = divmod(i - 7, 300)
        if off == 0 and k < len(want):
            if kind == "distinct":
                j = rng.choice(n, want[k], replace=False)
            else:
                pairs = min(want[k] // 2, two.size)
                j = np.concatenate([rng.choice(two, pairs, replace=False),
                                    rng.choice(one, want[k] - 2 * pairs, replace=False),
                                    rng.choice(np.flatnonzero(length == 0), 40, replace=False)])
        else:
            j = np.unique(np.append(rng.integers(0, n, 3), i))
        rows.append(np.full(j.size, i))
        cols.append(np.sort(j))
    A = csr(np.concatenate(rows), np.concatenate(cols), (n, n), rng)
    return A, P, want


@pytest.mark.parametrize("longest", [8192, 8193])
@pytest.mark.parametrize("kind", ["distinct", "shared"])
def test_limits(kind, longest):
    from paper_2606_19251_amd import capi

    A, P, want = problem(kind, longest)
    count = products(A, P)
    assert set(want) <= set(count.tolist()) and count.max() == longest
    AP = (A @ P).tocsr()
    most = np.diff(AP.indptr).max()
    assert most == longest if kind == "distinct" else most < 1500
    # the second product meets the same limits where a coarse point restricts one long row alone
    if kind == "distinct":
        assert set(want) <= set(products(P.T.tocsr(), AP).tolist())
    got = capi.amgg_galerkin_device(0, A.shape[0], P.shape[1], *dev(A), *dev(P))
    ref = amg.galerkin(A, P)
    for g, r in zip(got, (ref.indptr, ref.indices, ref.data)):
        g, r = g.cpu().numpy(), np.ascontiguousarray(r)
        assert np.array_equal(g.view(np.uint64), r.view(np.uint64)) if g.dtype == np.float64 else np.array_equal(g, r)
