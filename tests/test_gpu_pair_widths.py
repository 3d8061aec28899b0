"""Which levels take the paired passes (the padded widths in use against the rule, computed here from the
matrices), and every kernel of theirs: rows of R in 8, 16 and 32 places with rows of A in 16, 32 and 64 for
the residual with restriction, rows of A in 8, 16, 32 and 64 for the prolongation, rows of P in more than
four. Ragged rows, sizes that are no multiple of a workgroup's rows; both sides of the limits on
widths, rows and repeated work. The sums keep their order: bit for bit the separate passes (fusion off)."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MAX_ROWS, MAX_SLOTS, MAX_WORK, MAX_A, MAX_R = 32768, 1 << 19, 1 << 20, 64, 32


def hierarchy(n, half, p, nc, thin=0.0):
    """Two levels: a band matrix of 2 half + 1 entries a row (a share `thin` of its couplings taken out) and a
    prolongation of p entries a row over nc columns, dealt in turn."""
    from paper_2606_19251_amd.solver import HostHierarchy, HostLevel

    rng = np.random.default_rng(n + half)
    i = np.repeat(np.arange(n), half)
    j = i + np.tile(np.arange(1, half + 1), n)
    keep = (j < n) & ((rng.random(j.size) >= thin) | (j == i + 1))
    i, j = i[keep], j[keep]
    w = rng.uniform(0.2, 1.0, i.size)
    A = sp.coo_matrix((np.r_[-w, -w], (np.r_[i, j], np.r_[j, i])), shape=(n, n)).tocsr()
    A = (A + sp.diags(0.1 - np.asarray(A.sum(axis=1)).ravel())).tocsr()
    A.sort_indices()
    rows = np.repeat(np.arange(n), p) if p >= 1 else np.arange(0, n, round(1 / p))
    cols = np.arange(rows.size) % nc
    P = sp.csr_matrix((rng.uniform(0.2, 1.0, rows.size), (rows, cols)), shape=(n, nc))
    P.sort_indices()
    C = (P.T @ A @ P).tocsr()
    C.sort_indices()
    lv = lambda M, **kw: HostLevel(M.shape[0], M.indptr.astype(np.int32), M.indices.astype(np.int32), M.data, **kw)
    h = HostHierarchy([lv(A, p_ncols=nc, p_rowptr=P.indptr.astype(np.int32), p_col=P.indices.astype(np.int32),
                          p_val=P.data), lv(C)], False)
    return h, A, P


def expected(A, P):
    n, nc = P.shape
    longest = lambda M: int(np.diff(M.indptr).max())
    cap = lambda rows, nz, widest: min(widest, (5 * nz // (2 * rows) + 7) // 4 * 4) if n <= MAX_ROWS else 0
    R = P.T.tocsr()
    caps = [cap(n, A.nnz, MAX_A), cap(n, P.nnz, MAX_A), cap(nc, P.nnz, MAX_R)]
    w = [max(4, (longest(M) + 3) // 4 * 4) for M in (A, P, R)]
    fits = all(a <= b for a, b in zip(w, caps)) and n * w[0] <= MAX_SLOTS and nc * w[2] * w[0] <= MAX_WORK
    return w if fits else [0, 0, 0]


# n, half band, entries of P a row, coarse rows, thinned share -> widths of A, P, R (0: separate passes)
CASES = [
    # rows of R: 4, 8 | 9..16 | 17..32 with rows of A up to 16 (of them 4 and 8: eight lanes a row)
    ((963, 1, 2, 486, 0.0), [4, 4, 4]), ((961, 3, 2, 242, 0.3), [8, 4, 8]), ((960, 5, 2, 240, 0.0), [12, 4, 8]),
    ((957, 7, 2, 150, 0.2), [16, 4, 16]), ((960, 4, 2, 60, 0.0), [12, 4, 32]), ((965, 7, 2, 100, 0.0), [16, 4, 20]),
    # rows of A up to 32
    ((959, 8, 2, 242, 0.1), [20, 4, 8]), ((960, 12, 2, 150, 0.0), [28, 4, 16]), ((962, 15, 2, 62, 0.3), [32, 4, 32]),
    # rows of A up to 64
    ((960, 16, 2, 480, 0.0), [36, 4, 4]), ((967, 20, 2, 130, 0.2), [40, 4, 16]), ((960, 31, 2, 60, 0.0), [64, 4, 32]),
    # rows of P in 8 and 12 places
    ((700, 3, 6, 210, 0.0), [8, 8, 20]), ((701, 9, 10, 350, 0.2), [20, 12, 24]),
    # one place too many: A of 65 entries, R of 33
    ((960, 32, 2, 60, 0.0), None), ((960, 3, 2, 58, 0.0), None),
    # rows of the level, where nothing else decides
    ((32768, 1, 1 / 32, 1024, 0.0), [4, 4, 4]), ((32769, 1, 1 / 32, 1024, 0.0), None),
    # repeated work: 910 rows of R in 32 places, of A in 36, stay below 2^20, 911 do not
    ((14560, 17, 2, 910, 0.0), [36, 4, 32]), ((14563, 17, 2, 911, 0.0), None),
    # places of A: 2^19 and one row more
    ((32768, 7, 1 / 64, 512, 0.0), [16, 4, 4]), ((21846, 10, 1 / 64, 342, 0.0), None),
]


def test_cases_reach_every_kernel():
    took = [w for _, w in CASES if w]
    place = lambda v, limits: next(m for m in limits if v <= m)
    down = {(place(w[2], (8, 16, 32)), place(w[0], (16, 32, 64))) for w in took}
    assert down == {(r, a) for r in (8, 16, 32) for a in (16, 32, 64)}
    assert {place(w[0], (8, 16, 32, 64)) for w in took} == {8, 16, 32, 64}


@pytest.mark.parametrize("case,widths", CASES)
def test_pairs_bitwise(case, widths):
    from paper_2606_19251_amd import capi
    from paper_2606_19251_amd.solver import DeviceSolver

    h, A, P = hierarchy(*case)
    want = expected(A, P)
    assert want == (widths or [0, 0, 0])
    ds = DeviceSolver(h)
    ds.set_jacobi()
    assert capi.amgg_pair_widths(ds.ctx, 0) == want
    rng = np.random.default_rng(1)
    f, u0 = (torch.from_numpy(rng.standard_normal(A.shape[0])).cuda() for _ in range(2))
    for precision in (64, 32):
        for nu1, nu2 in ((1, 1), (2, 2)):
            out = []
            for fused in (True, False):
                ds.set_fusion(fused)
                assert capi.amgg_pair_widths(ds.ctx, 0) == (want if fused else [0, 0, 0])
                u = u0.clone()
                ds.vcycle(f, u, nu1, nu2, precision)
                out.append(u.cpu().numpy())
            assert np.isfinite(out[0]).all()
            assert np.array_equal(out[0].view(np.uint64), out[1].view(np.uint64)), (precision, nu1, nu2)
    ds.close()
