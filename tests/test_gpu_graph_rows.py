"""The all-pairs edge test with few rows (rows of A a lane holds: 1, 4, 8 or 16) and
with most pairs joined, whose out-degrees are sums over every block of a row."""
import types

import numpy as np
import pytest

from tests.test_gpu_graph_edges import _adjacency

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31])
@pytest.mark.parametrize("n,bound", [(17, 0.5), (130, 20.0), (401, 1.0), (401, 20.0)])
def test_few_rows(m, n, bound):
    import torch
    from paper_2411_13507_amd.api import GraphGPU
    rng = np.random.default_rng(1000 * m + n)
    V = rng.uniform(0, 6, (n, 3))
    a = rng.standard_normal((m, 3))
    F1, F2, G = -a, a + 0.02 * rng.standard_normal((m, 3)), bound * rng.uniform(0.5, 1.5, m)
    adj, sure = _adjacency(V, F1, F2, G)
    words, deg = GraphGPU(types.SimpleNamespace(F1=F1, F2=F2, G=G), n).run(torch.as_tensor(V, device="cuda"))
    bits = np.unpackbits(words.cpu().numpy().view(np.uint8), axis=1, bitorder="little")
    got = bits[:, :n].astype(bool)
    assert np.array_equal(got[sure], adj[sure]) and sure.mean() > 0.99
    assert not bits[:, n:].any() and np.array_equal(deg.cpu().numpy(), got.sum(1))
    assert bound < 20.0 or got.mean() > 0.8
