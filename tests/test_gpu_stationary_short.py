"""A stationary solve enqueues no iteration blindly: one that ends within its first iterations leaves the whole
workspace, byte for byte, as the same solve limited to that many iterations does (an iteration run
past the converging one would leave its iterate and its scalars there)."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("graphs", [True, False])
@pytest.mark.parametrize("n,tol", [(18, 1e-8), (18, 0.3), (70, 0.1), (250, 0.3)])
def test_no_iteration_past_the_last(n, tol, graphs):
    from paper_2606_19251_amd import capi
    from paper_2606_19251_amd.solver import DeviceSolver, HostHierarchy

    A = W.grid5(n)
    ds = DeviceSolver(HostHierarchy.build(A.rowptr, A.col, A.val))
    ds.set_jacobi()
    b = torch.from_numpy(W.rhs_uniform(A.nrows, 3)).cuda()
    how = dict(outer=capi.AMGG_OUTER_STATIONARY, precision=64, tol=tol, graphs=graphs)
    iterations = ds.solve(b, **how)[2].iterations
    assert iterations <= 2
    out = []
    for maxit in (iterations, 500, iterations):
        x = torch.full_like(b, float("nan"))
        _, rc, info, _ = ds.solve(b, x, maxit=maxit, **how)
        torch.cuda.synchronize()
        assert rc == 0 and info.iterations == info.vcycles == iterations
        out.append((x, ds.ws.clone()))
    for x, ws in out[1:]:
        assert torch.equal(x, out[0][0]) and torch.equal(ws, out[0][1])
    ds.close()
