"""The dense inverse of the coarsest level around the panels' and wavefronts' edges: against numpy's inverse in
FP64, on well-conditioned matrices that need row exchanges, on one of equal pivots (ties go to the first
row), on the rank-one fix of an all-Neumann matrix and on singular ones, which are refused.

Both sides have an error of at most about n eps times the condition number (below 1e3 here), relative to
the inverse's largest entry."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _solver(M, singular=0):
    from paper_2606_19251_amd import capi

    n = M.shape[0]
    ptr = torch.arange(0, n * n + 1, n, dtype=torch.int32, device="cuda")
    col = torch.arange(n, dtype=torch.int32, device="cuda").repeat(n).contiguous()
    val = torch.from_numpy(np.ascontiguousarray(M.reshape(-1))).cuda()
    ctx = capi.amgg_create(0, 1)
    try:
        capi.amgg_load_level(ctx, 0, n, n * n, ptr.data_ptr(), col.data_ptr(), val.data_ptr())
        nbytes = capi.amgg_workspace_bytes(ctx)
        ws = torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")
        off = (-ws.data_ptr()) % 256
        st = torch.cuda.current_stream().cuda_stream
        capi.amgg_finalize(ctx, singular, ws.data_ptr() + off, nbytes, st)
        v = capi.amgg_level_view_get(ctx, 0)
        at = v.coarse_inv - ws.data_ptr()
        return ws[at:at + 8 * n * n].view(torch.float64).cpu().numpy().reshape(n, n)
    finally:
        capi.amgg_destroy(ctx)


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 64, 65, 96, 127, 129, 255, 257, 500, 513, 1023, 1024, 1025])
def test_inverse_with_exchanges(n):
    rng = np.random.default_rng(n)
    M = rng.standard_normal((n, n)) / np.sqrt(n)
    M[np.arange(n), rng.permutation(n)] += 3.0  # the largest entries lie off the diagonal
    M[np.arange(n), np.arange(n)] = np.abs(np.diag(M)) + 1e-3  # (a level's diagonal is positive)
    got, ref = _solver(M), np.linalg.inv(M)
    cond = np.linalg.cond(M)
    assert cond < 1e3
    assert np.abs(got - ref).max() <= max(n, 8) * 2.3e-16 * cond * np.abs(ref).max()


@pytest.mark.parametrize("n", [3, 40, 130])
def test_equal_pivots_and_rank_one_fix(n):
    T = 2 * np.eye(n) - np.eye(n, k=1) - np.eye(n, k=-1)
    H = np.where(np.add.outer(np.arange(n), np.arange(n)) % 2 == 0, 1.0, -0.5) + n * np.eye(n)
    for M in (T, H):
        ref = np.linalg.inv(M)
        assert np.abs(_solver(M) - ref).max() <= max(n, 8) * 2.3e-16 * np.linalg.cond(M) * np.abs(ref).max()
    N = T.copy()
    N[0, 0] = N[-1, -1] = 1.0
    ref = np.linalg.inv(N + np.trace(N) / n / n)
    assert np.abs(_solver(N, 1) - ref).max() <= max(n, 8) * 2.3e-16 * np.linalg.cond(N + np.trace(N) / n / n) * np.abs(ref).max()


@pytest.mark.parametrize("n", [2, 40, 200])
def test_singular_matrix_is_refused(n):
    M = 2 * np.eye(n)
    M[0, n - 1] = M[n - 1, 0] = 2.0  # equal rows: an exactly zero pivot at the end
    with pytest.raises(Exception, match="singular"):
        _solver(M)
