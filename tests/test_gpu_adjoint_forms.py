"""The V-cycle adjoint at the edges of its forms: smallest and largest degree, sweeps on one side only, and
the second cycle of a run from zero; against the oracle's complex-step gradient.

The first cycle of a run without an initial guess takes its first step without the residual pass (forward
and back), the gradient kernel has one instance per degree, and the level's right-hand-side adjoint starts
at its last step back, or is cleared where there is none. Both sides compute in FP64 over the same levels;
the bounds are those of the complex-step comparison at degrees 2 and 3.
"""
import numpy as np
import pytest

import workloads as W
from oracle import amg, grad

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

_cache = {}


def _problem():
    if not _cache:
        from paper_2606_19251_amd.solver import DeviceSolver, HostHierarchy

        A = W.delaunay_p1(W.gmm_points(700, 5))
        f = W.rhs_uniform(A.nrows, 9, zero_mean=True)
        kw = dict(max_levels=10, max_coarse=40)
        An, fn, sing = amg.normalize(A, f)
        _cache["p"] = (fn, amg.setup(An, singular=sing, **kw), DeviceSolver(HostHierarchy.build(A.rowptr, A.col, A.val, **kw), 0))
    return _cache["p"]


@pytest.mark.parametrize("degree", [1, 4])
@pytest.mark.parametrize("nu,nvc", [((1, 1), 1), ((1, 0), 1), ((0, 1), 1), ((0, 2), 2), ((2, 0), 2), ((1, 1), 3)])
def test_adjoint_forms(degree, nu, nvc):
    from paper_2606_19251_amd import capi

    f, ho, ds = _problem()
    assert ho.nlevels >= 3
    diag, off = [0.6, 0.01, -0.001, 0.0001, 0.00001], [0.12, 0.01, -0.001, 0.0001]
    base = np.array(diag[: degree + 1] + off[:degree])
    c = base * (1 + 0.05 * np.random.default_rng(degree).standard_normal((ho.nlevels, base.size)))
    ds.set_coeffs(c, degree)
    fd = torch.from_numpy(f).cuda()
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    g = torch.zeros(ds.nlevels, base.size, dtype=torch.float64, device="cuda")
    capi.amgg_vcycle_loss_adjoint(ds.ctx, nu[0], nu[1], 64, nvc, fd.data_ptr(), 0, loss.data_ptr(), g.data_ptr(),
                                  ds.stream)
    torch.cuda.synchronize()
    ref_loss = grad.vcycle_loss(ho, c, degree, f, None, nvc, *nu)
    ref = grad.grad_complex_step(ho, c, degree, f, None, nvc, *nu)
    assert abs(loss.item() - ref_loss) <= 1e-11 * max(1.0, abs(ref_loss))
    assert np.abs(g.cpu().numpy() - ref).max() <= 1e-9 * np.abs(ref).max()
