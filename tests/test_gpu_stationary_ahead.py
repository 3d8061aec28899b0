"""The stationary iteration runs up to two iterations ahead of the one the host inspects: whatever stops it
(the tolerance, the limit, stagnation, divergence), the result is the iterate of the iteration it stopped
at. Histories and iterates are compared bit for bit between runs stopped at different limits, with and
without graphs, and each history entry with the residual of the returned iterate on the host (rounding
of one FP64 product: 1e-10 relative to the right-hand side)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def solver(n=70):
    from paper_2606_19251_amd.solver import DeviceSolver, HostHierarchy

    A = W.grid5(n)
    return A, DeviceSolver(HostHierarchy.build(A.rowptr, A.col, A.val))


def solve(ds, b, **kw):
    from paper_2606_19251_amd import capi

    x, rc, info, hist = ds.solve(b, outer=capi.AMGG_OUTER_STATIONARY, precision=64, history_cap=400, **kw)
    return x.cpu().numpy(), rc, info, np.array(hist)


def relres(A, x, b):
    return np.linalg.norm(b - A.to_scipy() @ x) / np.linalg.norm(b)


@pytest.mark.parametrize("nu", [1, 2])
def test_limits_are_prefixes(nu):
    A, ds = solver()
    ds.set_jacobi()
    bh = W.rhs_uniform(A.nrows, 3)
    b = torch.from_numpy(bh).cuda()
    full = solve(ds, b, nu1=nu, nu2=nu, tol=1e-8)
    assert full[1] == 0 and full[2].iterations == len(full[3]) - 1
    assert abs(relres(A, full[0], bh) - full[3][-1]) <= 1e-10
    for graphs in (True, False):
        for k in (1, 2, 3, 4, 5, full[2].iterations - 1):
            x, rc, info, hist = solve(ds, b, nu1=nu, nu2=nu, tol=1e-8, maxit=k, graphs=graphs)
            assert rc == 1 and info.iterations == k and info.vcycles == k
            assert np.array_equal(hist, full[3][:k + 1])
            assert abs(relres(A, x, bh) - hist[-1]) <= 1e-10
        again = solve(ds, b, nu1=nu, nu2=nu, tol=1e-8, graphs=graphs)
        assert np.array_equal(again[0], full[0]) and np.array_equal(again[3], full[3])
    ds.close()


@pytest.mark.parametrize("omega,status", [(1e-7, 3), (3.0, 2)])  # stagnates; diverges
def test_stops_at_the_inspected_iterate(omega, status):
    A, ds = solver(40)
    ds.set_jacobi(omega)
    bh = W.rhs_uniform(A.nrows, 4)
    b = torch.from_numpy(bh).cuda()
    kw = dict(tol=1e-8, div_factor=10.0, stag_window=4, stag_ratio=0.99)
    x, rc, info, hist = solve(ds, b, fallback=False, **kw)
    assert rc == status and info.iterations == len(hist) - 1
    assert abs(relres(A, x, bh) - hist[-1]) <= 1e-10 * max(1.0, hist[-1])
    x2, rc2, info2, hist2 = solve(ds, b, fallback=True, **kw)  # omega-Jacobi goes on from that iterate
    assert rc2 == 0 and info2.fell_back == 1 and np.array_equal(hist2[:len(hist)], hist)
    assert relres(A, x2, bh) <= 1.01e-8
    ds.close()
