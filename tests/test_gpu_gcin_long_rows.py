"""Graph batches with rows of more entries than a tile's map holds: hub rows at the start, in the middle and at
the end of a tile and in its partial last one, rows past the limit of the map by one entry, against the oracle's
forward pass in FP64 (FP32 network: the tolerance of the other forward tests)."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import gcin as OG

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def hub_graph(n, hubs, k):
    """Path graph whose rows `hubs` are coupled to k nodes each."""
    rng = np.random.default_rng(n + k)
    i, j = [np.arange(n - 1)], [np.arange(1, n)]
    for h in hubs:
        t = rng.choice(np.setdiff1d(np.arange(n), [h]), k, replace=False)
        i.append(np.full(t.size, h))
        j.append(t)
    i, j = np.concatenate(i), np.concatenate(j)
    key = np.unique(np.minimum(i, j).astype(np.int64) * n + np.maximum(i, j))
    i, j = key // n, key % n
    w = rng.uniform(0.2, 1.0, i.size)
    A = sp.coo_matrix((np.r_[-w, -w], (np.r_[i, j], np.r_[j, i])), shape=(n, n)).tocsr()
    A = (A + sp.diags(0.1 - np.asarray(A.sum(axis=1)).ravel())).tocsr()
    A.sort_indices()
    return A


# the map holds 4096 entries of a tile's 64 rows
CASES = [(5000, [0], 4900), (5000, [63], 4900), (5000, [2500], 4500), (4999, [4998], 4900), (4481, [4479, 4480], 4300),
         (6000, [64, 127, 130], 5000), (4200, [100], 3900), (4200, [100], 4100)]


@pytest.mark.parametrize("n,hubs,k", CASES)
@pytest.mark.parametrize("hidden", [32, 64])
def test_hub_rows(n, hubs, k, hidden):
    from paper_2606_19251_amd import capi
    from paper_2606_19251_amd import gcin as G

    dev = torch.device("cuda", 0)
    mats = [hub_graph(n, hubs, k), hub_graph(70, [69], 60)]
    graphs = [tuple(torch.from_numpy(t).cuda() for t in (A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data))
              for A in mats]
    batch = G.GraphBatch(graphs, dev, hidden)
    flat = G.init_flat(2, 5, hidden=hidden)
    out = batch.forward(torch.from_numpy(flat).to(dev), 2, capi.GCIN_FP32).cpu().numpy()
    ref = OG.forward_np(G.unpack(flat, 2, hidden), mats, 2)
    assert np.abs(out - ref).max() <= 1e-4 * np.abs(ref).max()
    batch.close()


@pytest.mark.parametrize("n,hubs,k", [(3000, [0], 2900), (3000, [1500], 600), (3000, [17, 18, 19], 1500),
                                      (3000, [16, 20, 24, 28], 1500), (2999, [2998], 2000)])
@pytest.mark.parametrize("hidden", [32, 64])
def test_hub_rows_backward(n, hubs, k, hidden):
    """Hub rows alone in their wavefront's rows, several in one group of four, one in each group: the gradient
    against the oracle's in FP64 (FP32 network), and the same bits from run to run."""
    from paper_2606_19251_amd import capi
    from paper_2606_19251_amd import gcin as G

    dev = torch.device("cuda", 0)
    mats = [hub_graph(n, hubs, k), hub_graph(130, [100], 60)]
    graphs = [tuple(torch.from_numpy(t).cuda() for t in (A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data))
              for A in mats]
    batch = G.GraphBatch(graphs, dev, hidden)
    flat = G.init_flat(2, 5, hidden=hidden)
    P = torch.from_numpy(flat).to(dev)
    batch.forward(P, 2, capi.GCIN_FP32)
    w = np.random.default_rng(3).standard_normal((2, 5))
    d = torch.from_numpy(w.astype(np.float32)).to(dev)
    g = batch.backward(P, d, 2, capi.GCIN_FP32)
    assert torch.equal(g, batch.backward(P, d, 2, capi.GCIN_FP32))
    ref = G.pack(OG.gradient(G.unpack(flat, 2, hidden), mats, w.astype(np.float32).astype(np.float64), 2), 2)
    g, ref = g.cpu().numpy().astype(np.float64), np.asarray(ref, np.float64)
    assert np.linalg.norm(g - ref) <= 1e-3 * np.linalg.norm(ref)
    batch.close()
