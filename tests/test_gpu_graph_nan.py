"""A row without a number in a whole tile of nodes rules out the tile's pairs: a
NaN bound joins nothing, and a tile that holds nothing but NaN nodes has no edges.
Sizes at one tile, its remainder and several tiles, row counts at the row chunks."""
import types

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 64, 65, 200])
@pytest.mark.parametrize("m,dim", [(1, 3), (16, 6), (33, 2)])
@pytest.mark.parametrize("where", ["G", "F1", "F2", "V"])
def test_no_edges_through_nan(n, m, dim, where):
    import torch
    from paper_2411_13507_amd.api import GraphGPU, graph_run_noalloc
    rng = np.random.default_rng(n + m)
    V = rng.uniform(0, 1, (n, dim))
    F1, F2, G = rng.standard_normal((m, dim)), rng.standard_normal((m, dim)), np.full(m, 1e3)   # joins every pair
    g = types.SimpleNamespace(F1=F1, F2=F2, G=G)
    full = n * (n - 1)
    if where == "V":
        t = (n - 1) // 64 * 64                      # the last tile
        V[t:] = np.nan
        full = t * (t - 1)
    else:
        getattr(g, where)[m // 2] = np.nan
        full = 0
    words, deg = GraphGPU(g, n).run(torch.as_tensor(V, device="cuda"))
    assert int(deg.sum()) == full
    assert np.unpackbits(words.cpu().numpy().view(np.uint8)).sum() == full
    w2, d2 = graph_run_noalloc(*(torch.as_tensor(x, device="cuda") for x in (g.F1, g.F2, g.G, V)))
    assert torch.equal(words, w2) and torch.equal(deg, d2)
