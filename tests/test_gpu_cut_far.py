"""Far pairs of the graph cut are decided from the edge's centroid and reach;
the others go through a list.  Sizes at the edges of its tiles (4 edges per
thread, 1,024 edges and 8 obstacles per block, 1,024 listed pairs per block)
and inputs that the far test has to leave to the general path, against Alg. 2
in NumPy (steps 1 and 2) and the library's own count of the pairs of step 3."""
import types

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _steps(P, lo, hi):
    """Deciding step per (box, edge) in FP64 and the margin of step 2 (how far
    the nearest control point lies beyond the plane, relative to its terms)."""
    c = P.mean(1)
    inside = ((P[None] >= lo[:, None, None]) & (P[None] <= hi[:, None, None])).all(-1).any(-1)
    n = c[None] - np.clip(c[None], lo[:, None], hi[:, None])
    off = np.where(n > 0, n * hi[:, None], n * lo[:, None]).sum(-1)
    gap = (n[:, :, None] * P[None]).sum(-1).min(-1) - off
    mag = np.abs(n).sum(-1) * np.maximum(np.abs(P).max(), 1.0)
    beyond = (n != 0).any(-1) & (gap > 0)
    return np.where(inside, 1, np.where(beyond, 2, 3)), np.abs(gap) > 1e-12 * mag


def _box_rows(lo, hi):
    A = np.concatenate([np.eye(3), -np.eye(3)])
    off = 6 * np.arange(len(lo) + 1)
    return off.astype(np.int32), np.tile(A, (len(lo), 1)), np.concatenate([hi, -lo], 1).reshape(-1)


@pytest.mark.parametrize("n_edges,n_box", [(1, 1), (3, 7), (4, 8), (5, 9), (1023, 8), (1024, 17), (1028, 3), (2051, 16)])
@pytest.mark.parametrize("length", [0.05, 0.6, 12.0])
def test_steps_and_counts(n_edges, n_box, length):
    import torch
    from paper_2411_13507_amd.api import CutGPU
    rng = np.random.default_rng(n_edges * 31 + n_box)
    a = rng.uniform(0, 10, (n_edges, 1, 3))
    P = a + length * rng.uniform(-0.5, 0.5, (n_edges, 6, 3))
    lo = rng.uniform(0, 9, (n_box, 3))
    hi = lo + rng.uniform(0.2, 1.5, (n_box, 3))
    off, A, b = _box_rows(lo, hi)
    prob = types.SimpleNamespace(box_lo=lo, box_hi=hi, degree=5, pob_off=off, pob_A=A, pob_b=b)
    g = CutGPU(prob, n_edges)
    want, sure = _steps(P, lo, hi)
    for _ in range(2):
        r = g.run(torch.as_tensor(P, device="cuda"))
        step, code, d2 = r.step.cpu().numpy(), r.code.cpu().numpy(), r.qp_dist2.cpu().numpy()
        for s in (step[:n_box], step[n_box:]):     # boxes, then the same boxes as six rows
            assert np.array_equal(s[sure], want[sure])
        assert g.qp_count() == int((step == 3).sum())
        assert np.array_equal(np.isnan(d2), step != 3)
        assert np.array_equal(code[step != 3], step[step != 3] == 2)
        assert np.array_equal(code[step == 3], d2[step == 3] > 0)
        assert np.array_equal(r.n_collide.cpu().numpy(), (code == 0).sum(0))
        # codes alone take the same route
        r2 = g.run(torch.as_tensor(P, device="cuda"), with_step=False, with_dist=False)
        assert torch.equal(r2.code, r.code) and torch.equal(r2.n_collide, r.n_collide)


def test_inputs_without_far_pairs():
    """A NaN or infinite control point, an unbounded box: the plane test of
    step 2 cannot hold there, so none of these pairs is decided by it unless
    the general test says so."""
    import torch
    from paper_2411_13507_amd.api import CutGPU
    P = np.full((4, 4, 3), 5.0) + 0.01 * np.arange(12).reshape(4, 1, 3)
    P[1, 2, 0] = np.nan
    P[2, 1, 1] = np.inf
    lo = np.array([[0.0, 0.0, 0.0], [-np.inf, 8.0, 8.0], [9.0, 9.0, 9.0]])
    hi = np.array([[1.0, 1.0, 1.0], [np.inf, 9.0, 9.0], [9.5, 9.5, 9.5]])
    g = CutGPU(types.SimpleNamespace(box_lo=lo, box_hi=hi, degree=3), 4)
    step = g.run(torch.as_tensor(P, device="cuda")).step.cpu().numpy()
    assert (step[[0, 2]][:, [0, 3]] == 2).all()       # plain far pairs
    assert (step[:, 1] == 3).all()                    # NaN point
    assert (step[1] == 3).all()                       # 0 * inf in the plane's offset
