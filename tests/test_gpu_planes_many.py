"""Adjacent hyperplanes of so many nodes that a block is one wavefront, around the
node count where it becomes one."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [131_008, 131_009, 131_073])
@pytest.mark.parametrize("n_box", [8, 33])
def test_nearest_box(n, n_box):
    import torch
    from paper_2411_13507_amd.api import adjacent_hyperplanes
    g = torch.Generator(device="cuda").manual_seed(n + n_box)
    X = 10 * torch.rand(n, 3, dtype=torch.float64, device="cuda", generator=g)
    lo = 9 * torch.rand(n_box, 3, dtype=torch.float64, device="cuda", generator=g)
    hi = lo + 1.0
    idx, point, _ = adjacent_hyperplanes(X, lo, hi)
    c = torch.minimum(torch.maximum(X[:, None], lo), hi)
    d2 = ((X[:, None] - c) ** 2).sum(-1)
    best, want = d2.min(1)
    # (two boxes may hold a node, and rounding may order two near-equal distances either way)
    sure = (d2 <= best[:, None] * (1 + 1e-14)).sum(1) == 1
    assert sure.float().mean() > 0.8 and torch.equal(idx[sure].long(), want[sure])
    assert torch.equal(point, c[torch.arange(n, device="cuda"), idx.long()])
