"""GCIN batches at the edges of their 64-row tiles: graphs of one row less than, exactly and one row more
than whole tiles, with short rows, rows longer than a gather batch and rows whose tile overflows the
batch copy's entry map (more than 64 entries a row), alone and together, forward and backward against
the FP64 oracle. Tolerances are the network's at every size: FP32 1e-4 forward, 2e-3 and cosine
0.99999 backward; split BF16 1e-3 forward, 5e-2 and cosine 0.999 backward."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import gcin as OG

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SHAPES = [(5, 1), (63, 2), (64, 3), (65, 6), (127, 30), (128, 1), (129, 40), (191, 9), (1025, 4)]


def banded(n, half):
    rng = np.random.default_rng(n)
    half = min(half, n - 1)
    i = np.concatenate([np.arange(n - k) for k in range(1, half + 1)])
    j = np.concatenate([np.arange(k, n) for k in range(1, half + 1)])
    v = rng.uniform(0.2, 1.0, i.size) / half
    L = sp.coo_matrix((np.concatenate([-v, -v]), (np.concatenate([i, j]), np.concatenate([j, i]))), shape=(n, n)).tocsr()
    L = (L + sp.diags(-np.asarray(L.sum(axis=1)).ravel() + rng.uniform(0.1, 1.0, n))).tocsr()
    L.sort_indices()
    return L


def params(degree, hidden):
    from paper_2606_19251_amd import gcin as G

    p = OG.init_params(degree, 5, hidden=hidden)
    rng = np.random.default_rng(6)
    for l in range(4):
        p[f"norm{l}.beta"] = rng.uniform(-0.3, 0.6, hidden)
        p[f"norm{l}.gamma"] = rng.uniform(0.7, 1.3, hidden)
    p["mlp2.b"] = np.zeros(2 * degree + 1)
    p["mlp2.W"] *= 3.0
    flat = G.pack(p, degree)
    return flat, G.unpack(flat, degree, hidden)


@pytest.mark.parametrize("hidden,precision,tf,tb,cos", [(64, 0, 1e-4, 2e-3, 0.99999), (64, 2, 1e-3, 5e-2, 0.999),
                                                        (32, 0, 1e-4, 2e-3, 0.99999)])
@pytest.mark.parametrize("pick", [None, 0, 2, 3, 6])
def test_tiles_match_oracle(hidden, precision, tf, tb, cos, pick):
    from paper_2606_19251_amd import gcin as G

    dev = torch.device("cuda", 0)
    mats = [banded(n, h) for n, h in (SHAPES if pick is None else [SHAPES[pick]])]
    graphs = [tuple(torch.from_numpy(a).to(dev) for a in (m.indptr.astype(np.int32), m.indices.astype(np.int32), m.data))
              for m in mats]
    flat, p64 = params(2, hidden)
    P = torch.from_numpy(flat).to(dev)
    batch = G.GraphBatch(graphs, dev, hidden)
    ref = OG.forward_np(p64, mats, 2)
    out = batch.forward(P, 2, precision).cpu().numpy()
    assert np.abs(out - ref).max() <= tf * np.abs(ref).max()
    small = G.GraphBatch(graphs, dev, hidden, inference=True).forward(P, 2, precision).cpu().numpy()
    assert np.array_equal(small, out)
    w = np.random.default_rng(9).standard_normal(ref.shape)
    g = batch.backward(P, torch.from_numpy(w.astype(np.float32)).to(dev), 2, precision).cpu().numpy().astype(np.float64)
    gref = G.pack(OG.gradient(p64, mats, w, 2), 2).astype(np.float64)
    assert np.abs(g - gref).max() <= tb * np.abs(gref).max()
    assert g @ gref >= cos * np.linalg.norm(g) * np.linalg.norm(gref)
