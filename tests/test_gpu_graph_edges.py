"""The all-pairs edge test at the edges of its tiles: 64 start nodes per
wavefront, 16 end nodes per wavefront, 128 per block, 16 rows per chunk and 64
per bound, the dimensions with kernels of their own and the general one, and
nodes that are NaN (which violate no row)."""
import types

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _adjacency(V, F1, F2, G):
    """Bool [n, n] by the definition, and whether every row of the pair is
    clear of its bound by more than rounding."""
    A, B = V @ F1.T, V @ F2.T - G
    s = A[:, None] + B[None]
    adj = ~(s > 0).any(-1)
    np.fill_diagonal(adj, False)
    return adj, (np.abs(s) > 1e-12 * (1 + np.abs(A[:, None]) + np.abs(B[None]))).all(-1)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 400])
@pytest.mark.parametrize("m,dim", [(1, 3), (15, 3), (16, 6), (17, 2), (64, 3), (65, 6), (130, 12)])
def test_against_numpy(n, m, dim):
    import torch
    from paper_2411_13507_amd.api import GraphGPU, graph_run_noalloc
    rng = np.random.default_rng(1000 * n + 10 * m + dim)
    V = rng.uniform(0, 6, (n, dim))
    V = V[np.argsort(V[:, 0])]                     # far tiles to skip, and near ones
    a = rng.standard_normal((m, dim))
    F1, F2, G = -a, a + 0.02 * rng.standard_normal((m, dim)), rng.uniform(0.5, 3.0, m) * np.sqrt(dim)
    if n > 64:
        V[n // 2] = np.nan
    adj, sure = _adjacency(V, F1, F2, G)
    if n > 64:   # a NaN node's pairs depend on which tiles the bounds skip
        sure[n // 2] = sure[:, n // 2] = False
    g = GraphGPU(types.SimpleNamespace(F1=F1, F2=F2, G=G), n)
    Vd = torch.as_tensor(V, device="cuda")
    words, deg = g.run(Vd)
    bits = np.unpackbits(words.cpu().numpy().view(np.uint8), axis=1, bitorder="little")
    got = bits[:, :n].astype(bool)
    assert np.array_equal(got[sure], adj[sure])
    assert not bits[:, n:].any() and not got[np.arange(n), np.arange(n)].any()
    assert np.array_equal(deg.cpu().numpy(), got.sum(1))
    if n > 64:   # a NaN start node is joined at least to the other nodes of its own tile
        t = n // 2 // 64 * 64
        near = np.arange(t, min(t + 64, n))
        assert got[n // 2, near[near != n // 2]].all()
    dev = [torch.as_tensor(x, device="cuda") for x in (F1, F2, G)]
    w2, d2 = graph_run_noalloc(*dev, Vd)
    assert torch.equal(words, w2) and torch.equal(deg, d2)
