"""Batches whose layer arrays exceed 4 GiB, where the gathers take 64-bit byte offsets: copies of one graph, whose
coefficients do not depend on what else is in the batch (bit for bit those of the graph alone), and the
gradient through the last copy, whose rows lie past the limit, against the graph's own. The batch's sums of the
parameter gradients only group the same terms differently: FP32 sums of up to 33 tiles' products a
workgroup, a few of 2^-24 each, so 1e-5 of the gradient's norm."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def graph():
    """1000 x 1001 grid with random couplings (no two rows alike, and no multiple of a power of two)."""
    rng = np.random.default_rng(2)
    nx, ny = 1000, 1001
    idx = np.arange(nx * ny).reshape(nx, ny)
    i = np.r_[idx[:-1].ravel(), idx[:, :-1].ravel()]
    j = np.r_[idx[1:].ravel(), idx[:, 1:].ravel()]
    w = rng.uniform(0.2, 1.0, i.size)
    A = sp.coo_matrix((np.r_[-w, -w], (np.r_[i, j], np.r_[j, i])), shape=(idx.size, idx.size)).tocsr()
    A = (A + sp.diags(0.05 - np.asarray(A.sum(axis=1)).ravel())).tocsr()
    A.sort_indices()
    return tuple(torch.from_numpy(t).cuda() for t in (A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data))


@pytest.mark.parametrize("hidden,precision", [(64, "GCIN_FP32"), (64, "GCIN_BF16"), (64, "GCIN_BF16X3"), (32, "GCIN_FP32")])
def test_offsets_past_4_gib(hidden, precision):
    from paper_2606_19251_amd import capi
    from paper_2606_19251_amd import gcin as G

    precision = getattr(capi, precision)
    dev = torch.device("cuda", 0)
    g = graph()
    n = g[0].numel() - 1
    copies = 2 ** 32 // (4 * hidden * n) + 1
    assert (copies - 1) * n * hidden * 4 < 2 ** 32 < copies * n * hidden * 4
    P = torch.from_numpy(G.init_flat(2, 11, hidden=hidden)).to(dev)
    one = G.GraphBatch([g], dev, hidden)
    many = G.GraphBatch([g] * copies, dev, hidden)
    c1, c = one.forward(P, 2, precision), many.forward(P, 2, precision)
    assert torch.isfinite(c1).all() and torch.equal(c, c1.expand_as(c))
    d = torch.zeros_like(c)
    d[-1] = torch.tensor([0.3, -1.0, 0.7, 0.2, -0.4], device=dev)
    want = one.backward(P, d[-1:].contiguous(), 2, precision).double()
    got = many.backward(P, d, 2, precision).double()
    assert want.norm() > 0 and (got - want).norm() <= 1e-5 * want.norm()
    one.close()
    many.close()
    del one, many
    torch.cuda.empty_cache()
