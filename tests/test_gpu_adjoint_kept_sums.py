"""Coefficient gradients of block-diagonal hierarchies, whose steps' sums are added up together: fewer, exactly
and more steps than are kept at a time, coefficient rows of their own and rows shared by a block's levels (where every
step is added by itself). Against the problems one by one and against the sum over the levels; FP64 sums
in another order: 1e-12 relative to the largest entry."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

POLY2 = np.array([0.6, 0.01, -0.001, 0.12, 0.01])


@pytest.mark.parametrize("nu,nvc", [((1, 0), 1), ((2, 2), 1), ((3, 2), 1), ((1, 1), 2), ((1, 2), 3)])
def test_kept_sums(nu, nvc):
    from paper_2606_19251_amd import capi
    from paper_2606_19251_amd.solver import DeviceSolver, HostHierarchy, block_diagonal

    mats = [W.grid5(20), W.delaunay_p1(W.gmm_points(900, 1)), W.grid5(33)]
    hiers = [HostHierarchy.build(A.rowptr, A.col, A.val, max_levels=4, max_coarse=30) for A in mats]
    H, offsets, rows, sing = block_diagonal(hiers)
    total = sum(h.nlevels for h in hiers)
    f = [torch.from_numpy(W.rhs_uniform(A.nrows, k, zero_mean=True)).cuda() for k, A in enumerate(mats)]

    def run(blocks, nrows):
        ds = DeviceSolver(H, 0, blocks=blocks)
        ds.set_coeffs(POLY2, 2)
        loss = torch.zeros(len(mats), dtype=torch.float64, device="cuda")
        g = torch.full((nrows, 5), 7.0, dtype=torch.float64, device="cuda")
        cat = torch.cat(f)
        capi.amgg_vcycle_loss_adjoint_blocks(ds.ctx, nu[0], nu[1], 64, nvc, cat.data_ptr(), 0, loss.data_ptr(),
                                             g.data_ptr(), nrows, ds.stream)
        torch.cuda.synchronize()
        return loss.cpu().numpy(), g.cpu().numpy()

    loss, g = run((offsets, rows, sing), total)
    first = np.cumsum([0] + [h.nlevels for h in hiers])
    for p, h in enumerate(hiers):
        ds = DeviceSolver(h, 0)
        ds.set_coeffs(POLY2, 2)
        l1 = torch.zeros(1, dtype=torch.float64, device="cuda")
        g1 = torch.zeros(h.nlevels, 5, dtype=torch.float64, device="cuda")
        capi.amgg_vcycle_loss_adjoint(ds.ctx, nu[0], nu[1], 64, nvc, f[p].data_ptr(), 0, l1.data_ptr(), g1.data_ptr(), ds.stream)
        torch.cuda.synchronize()
        ref = g1.cpu().numpy()
        assert abs(l1.item() - loss[p]) <= 1e-12 * max(1.0, abs(loss[p]))
        assert np.abs(g[first[p]:first[p + 1]] - ref).max() <= 1e-12 * np.abs(ref).max()
    shared = [np.where(np.asarray(r) >= 0, np.arange(len(mats)), -1).astype(np.int32) for r in rows]
    loss2, gs = run((offsets, shared, sing), len(mats))
    assert np.array_equal(loss2, loss)
    for p in range(len(mats)):
        want = g[first[p]:first[p + 1]].sum(axis=0)
        assert np.abs(gs[p] - want).max() <= 1e-12 * np.abs(g[first[p]:first[p + 1]]).max()
