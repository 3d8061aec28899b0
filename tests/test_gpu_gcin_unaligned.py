"""Parameters, incoming gradients and results that start at any float: a run on views one float into larger
tensors gives bitwise what a run on tensors of their own gives (the kernels read parameters by 16 bytes)."""
import numpy as np
import pytest

import workloads as W
from oracle import gcin as OG

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("hidden,precision", [(64, 0), (64, 1), (64, 2), (32, 0)])
def test_views_at_odd_offsets(hidden, precision):
    from paper_2606_19251_amd import gcin as G

    dev = torch.device("cuda", 0)
    mats = [W.grid5(9), W.grid5(20)]
    graphs = [tuple(torch.from_numpy(np.ascontiguousarray(a)).to(dev) for a in (m.rowptr, m.col, m.val)) for m in mats]
    flat = torch.from_numpy(G.pack(OG.init_params(2, 3, hidden=hidden), 2)).to(dev)
    w = torch.from_numpy(np.random.default_rng(1).standard_normal((2, 5)).astype(np.float32)).to(dev)
    res = []
    for off in (0, 1, 3):
        P, dc = torch.zeros(flat.numel() + 8, device=dev), torch.zeros(w.numel() + 8, device=dev)
        P, dc = P[off:off + flat.numel()], dc[off:off + w.numel()].view_as(w)
        P.copy_(flat)
        dc.copy_(w)
        batch = G.GraphBatch(graphs, dev, hidden)
        out = batch.forward(P, 2, precision).clone()
        res.append((out, batch.backward(P, dc, 2, precision).clone()))
    assert torch.isfinite(res[0][1]).all() and res[0][1].abs().max() > 0
    for out, g in res[1:]:
        assert torch.equal(out, res[0][0]) and torch.equal(g, res[0][1])
