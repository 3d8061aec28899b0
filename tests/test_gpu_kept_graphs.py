"""Captured solve graphs over many right-hand sides, all held alive: the stationary iteration's graphs know no
address of the caller's, so their number does not grow with the tensors passed, and every solution is the one
of launches without graphs, bit for bit (the same kernels on the same values)."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_stationary_graphs_do_not_grow_with_the_right_hand_sides():
    from paper_2606_19251_amd import capi
    from paper_2606_19251_amd.solver import DeviceSolver, HostHierarchy

    A = W.grid5(40)  # Dirichlet: the right-hand side is not projected
    ds = DeviceSolver(HostHierarchy.build(A.rowptr, A.col, A.val))
    ds.set_jacobi()
    assert not ds.hier.singular
    bs = [torch.from_numpy(W.rhs_uniform(A.nrows, s)).cuda() for s in range(12)]
    xs = [torch.empty_like(b) for b in bs]
    kept = []
    for b, x in zip(bs, xs):
        _, rc, _, _ = ds.solve(b, x, outer=capi.AMGG_OUTER_STATIONARY, precision=64, tol=1e-8)
        assert rc == 0
        kept.append(capi.amgg_kept_graphs(ds.ctx))
    assert kept == [kept[0]] * len(kept)
    for b, x in zip(bs, xs):
        y, rc, _, _ = ds.solve(b, outer=capi.AMGG_OUTER_STATIONARY, precision=64, tol=1e-8, graphs=False)
        assert rc == 0 and torch.equal(x, y)
    ds.close()


@pytest.mark.parametrize("outer,precision", [("ir", 32), ("ir", 64), ("fcg", 32), ("fcg", 64)])
def test_kept_graphs_are_bounded(outer, precision):
    """Refinement and flexible CG capture the caller's x (and b): the oldest graphs go, and a tensor whose
    graphs are gone is solved again as before."""
    from paper_2606_19251_amd import capi
    from paper_2606_19251_amd.solver import DeviceSolver, HostHierarchy

    A = W.grid5(40)
    ds = DeviceSolver(HostHierarchy.build(A.rowptr, A.col, A.val))
    ds.set_jacobi()
    how = dict(outer={"ir": capi.AMGG_OUTER_IR, "fcg": capi.AMGG_OUTER_FCG}[outer], precision=precision, tol=1e-8)
    bs = [torch.from_numpy(W.rhs_uniform(A.nrows, s)).cuda() for s in range(90 if outer == "fcg" else 270)]
    xs = [torch.empty_like(b) for b in bs]
    kept = []
    for b, x in zip(bs, xs):
        assert ds.solve(b, x, **how)[1] == 0
        kept.append(capi.amgg_kept_graphs(ds.ctx))
    assert max(kept) == kept[-1] == 256
    for k in (0, 1, len(bs) - 1, 0):
        y = xs[k].clone()
        assert ds.solve(bs[k], xs[k], **how)[1] == 0 and torch.equal(xs[k], y)
        assert ds.solve(bs[k], graphs=False, **how)[1] == 0 and capi.amgg_kept_graphs(ds.ctx) == 256
        assert torch.equal(ds.solve(bs[k], graphs=False, **how)[0], y)
    ds.close()
