"""Row-wise Galerkin products: rows at the edges of every class of hash table (32, 128, 1024 and 8192
products, one more than each), rows without products, all rows of one class and rows of all classes
together, against the oracle's products bit for bit (the accumulation order is the same)."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import amg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev(M):
    return tuple(torch.from_numpy(a).cuda() for a in (M.indptr.astype(np.int32), M.indices.astype(np.int32), M.data))


def random_rows(counts, ncols, rng, diag):
    """CSR matrix with counts[i] entries in row i (and its diagonal, if asked for)."""
    rows, cols = [], []
    for i, c in enumerate(counts):
        k = rng.choice(ncols, size=min(c, ncols), replace=False)
        if diag:
            k = np.union1d(k, [i])
        rows.append(np.full(k.size, i))
        cols.append(np.sort(k))
    r, c = np.concatenate(rows).astype(np.int64), np.concatenate(cols).astype(np.int64)
    v = rng.uniform(-1.0, 1.0, r.size)
    M = sp.csr_matrix((v, (r, c)), shape=(len(counts), ncols))
    M.sort_indices()
    return M


@pytest.mark.parametrize("rows", ["short", "long", "all", "empty"])
def test_row_products_bitwise(rows):
    from paper_2606_19251_amd import capi

    rng = np.random.default_rng(3)
    n, nc = 700, 260
    counts = {"short": np.full(n, 4), "long": np.full(n, 90), "empty": np.where(np.arange(n) % 5 == 0, 3, 0),
              "all": np.resize([3, 15, 16, 17, 63, 64, 65, 200, 511, 512, 513, 699], n)}[rows]
    A = random_rows(counts, n, rng, True)
    # two entries a row, so that a row of A with k entries makes about 2 k products with P
    P = random_rows(np.full(n, 2), nc, rng, False)
    if rows == "empty":
        P = random_rows(np.where(np.arange(n) % 3 == 0, 2, 0), nc, rng, False)
    got = capi.amgg_galerkin_device(0, n, nc, *dev(A), *dev(P))
    ref = amg.galerkin(A, P)
    again = capi.amgg_galerkin_device(0, n, nc, *dev(A), *dev(P), chunk_products=100000)  # the expanding form
    for g, a, r in zip(got, again, (ref.indptr, ref.indices, ref.data)):
        g, a = g.cpu().numpy(), a.cpu().numpy()
        assert np.array_equal(g, a)
        assert np.array_equal(g.view(np.uint64) if g.dtype == np.float64 else g,
                              np.ascontiguousarray(r).view(np.uint64) if g.dtype == np.float64 else r)
