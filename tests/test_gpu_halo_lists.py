"""The halo lists that the fused smoothing steps run on, at the edges of what they hold: a block's halo
rows and halo entries at and one past their limits, several blocks and a partial last one, a single
block without a halo. Which levels have lists is compared with the rule on the host, and cycles on them
bit for bit with the separate passes (the sums keep their order)."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

HALO_ROWS, HALO_ENTRIES, FUSE_ROWS = 1024, 3072, 65536
POLY2 = np.array([0.6, 0.01, -0.001, 0.12, 0.01])


def _graph(n, i, j):
    key = np.unique(np.minimum(i, j) * np.int64(n) + np.maximum(i, j))
    i, j = key // n, key % n
    w = np.random.default_rng(n).uniform(0.2, 1.0, i.size)
    L = sp.coo_matrix((np.r_[-w, -w], (np.r_[i, j], np.r_[j, i])), shape=(n, n)).tocsr()
    L = (L + sp.diags(-np.asarray(L.sum(axis=1)).ravel() + 0.05)).tocsr()
    L.sort_indices()
    return L


def _star(leaves, ring, extra=0):
    """256 hubs (the first block), each with its share of the leaves; the first `ring` leaves form a ring among
    themselves, the first `extra` are linked once more; then a path of 4000 nodes, whose entries leave room for
    the others' halos (all of a level's halo entries together may not exceed its entries)."""
    leaf = 256 + np.arange(leaves)
    path = 256 + leaves + np.arange(4000)
    r, e = leaf[:ring], leaf[:extra]
    return _graph(path[-1] + 1, np.r_[np.arange(leaves) % 256, r, e, path[:-1]], np.r_[leaf, np.roll(r, -1), e + 2, path[1:]])


def _rows(n, nnz):
    for r in (256, 128, 64):
        if r * nnz / n <= 0.9 * 2048:
            return r
    for r in (256, 128, 64, 32):
        if r * nnz / n * 1.25 <= 4096:
            return r
    return 0


def _expected(ptr, col, n):
    rows = _rows(n, col.size) if n <= FUSE_ROWS else 0
    total = 0
    for r0 in range(0, n if rows else 0, rows):
        c = col[ptr[r0]:ptr[min(r0 + rows, n)]]
        out = np.unique(c[(c < r0) | (c >= r0 + rows)])
        ents = int((ptr[out + 1] - ptr[out]).sum())
        total += ents
        if out.size > HALO_ROWS or ents > HALO_ENTRIES:
            return 0
    return rows if total <= col.size else 0


CASES = {
    "rows_at_limit": (lambda: _star(1024, 0), 256),
    "rows_past_limit": (lambda: _star(1025, 0), 0),
    "entries_at_limit": (lambda: _star(768, 768), 256),
    "entries_past_limit": (lambda: _star(768, 768, extra=1), 0),
    "one_block": (lambda: _graph(200, np.arange(199), np.arange(1, 200)), 256),
    "whole_blocks": (lambda: _graph(1024, np.arange(1023), np.arange(1, 1024)), 256),
    "partial_block": (lambda: _graph(1025, np.r_[np.arange(1024), np.arange(900)], np.r_[np.arange(1, 1025), np.arange(900) + 125]), 256),
}


@pytest.mark.parametrize("name", list(CASES))
def test_halo_lists(name):
    from paper_2606_19251_amd.solver import DeviceSolver, HostHierarchy

    make, rows0 = CASES[name]
    A = make()
    n = A.shape[0]
    # (levels further down couple so weakly that the polynomial smoother overflows FP32 there)
    hier = HostHierarchy.build(A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data, max_levels=3, max_coarse=60)
    ds = DeviceSolver(hier)
    want = [_expected(np.asarray(L.rowptr), np.asarray(L.col), L.n) for L in hier.levels[:-1]]
    assert want[0] == rows0
    assert [ds.level_view(l)["fused_rows"] for l in range(hier.nlevels - 1)] == want
    ds.set_coeffs(POLY2, 2)
    rng = np.random.default_rng(3)
    f, u0 = torch.from_numpy(rng.standard_normal(n)).cuda(), torch.from_numpy(rng.standard_normal(n)).cuda()
    for precision in (64, 32):
        out = []
        for fused in (True, False):
            ds.set_fusion(fused)
            u = u0.clone()
            ds.vcycle(f, u, 2, 1, precision)
            out.append(u.cpu().numpy())
        assert np.array_equal(out[0].view(np.uint64), out[1].view(np.uint64)), precision
        assert np.isfinite(out[0]).all()
