"""Distances of the graph cut where faces of the simplex degenerate: control
points that coincide, or lie on a line, in a plane or anywhere on a lattice of
quarters, against boxes with lattice corners (some without thickness) that they
touch at a corner, an edge or a face, and against the same boxes as six rows.
Coordinates are exact, so distances are compared with the FP64 oracle at its own
1e-9 of the value and 1e-12 of the squared extent."""
import types

import numpy as np
import pytest

from oracle import cut as ocut

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank", [0, 1, 2, 3])
@pytest.mark.parametrize("p", [1, 3, 7])
def test_lattice_distances(gpu_available, p, rank):
    import torch
    from paper_2411_13507_amd.api import CutGPU
    rng = np.random.default_rng(10 * p + rank)
    n_e, n_o = 60, 12
    base = rng.integers(0, 24, (n_e, 1, 3)) / 4.0
    span = rng.integers(-4, 5, (n_e, rank, 3)) / 4.0
    P = base + np.einsum("eka,eac->ekc", rng.integers(0, 3, (n_e, p + 1, rank)).astype(float), span)
    lo = rng.integers(0, 20, (n_o, 3)) / 4.0
    hi = lo + rng.integers(1, 9, (n_o, 3)) / 4.0
    flat = hi.copy()
    flat[:3, 0] = lo[:3, 0]                         # boxes without thickness
    A = np.concatenate([np.eye(3), -np.eye(3)])
    off = (6 * np.arange(n_o + 1)).astype(np.int32)
    rows = np.concatenate([hi, -lo], 1).reshape(-1)
    prob = types.SimpleNamespace(box_lo=lo, box_hi=flat, degree=p, pob_off=off, pob_A=np.tile(A, (n_o, 1)), pob_b=rows)
    print(f"case: degree {p}, points of rank {rank}", flush=True)
    r = CutGPU(prob, n_e).run(torch.as_tensor(P, device="cuda"))
    step, code, d2 = r.step.cpu().numpy(), r.code.cpu().numpy(), r.qp_dist2.cpu().numpy()
    n3 = 0
    for o in range(2 * n_o):
        l, h = lo[o % n_o], (flat if o < n_o else hi)[o % n_o]
        for e in range(n_e):
            if step[o, e] != 3:
                continue
            n3 += 1
            want = ocut.cut_qp(P[e], l, h).dist2
            tol = 1e-12 * max(1.0, np.abs(P[e]).max()) ** 2
            assert abs(d2[o, e] - want) <= 1e-9 * want + tol, (o, e, d2[o, e], want)
            if want > tol:
                assert code[o, e] == 1
            elif o < n_o:
                assert code[o, e] == 0, (o, e, d2[o, e])
    assert n3 > 0 or rank == 0


@pytest.mark.parametrize("n_e,n_o", [(1, 4095), (3, 4100), (1030, 2100), (2, 270_000)])
def test_many_list_regions(gpu_available, n_e, n_o):
    """More list regions than the step kernel has wavefronts for (it then takes
    2 to 64 of them together), empty ones and full ones: deciding steps and counts
    against Alg. 2 in NumPy."""
    import torch
    from paper_2411_13507_amd.api import CutGPU
    from tests.test_gpu_cut_far import _steps
    rng = np.random.default_rng(n_o)
    P = rng.uniform(4, 6, (n_e, 1, 3)) + rng.uniform(-0.3, 0.3, (n_e, 4, 3))
    lo = rng.uniform(0, 9.5, (n_o, 3))
    lo[: n_o // 64] = 5 + 0.2 * rng.standard_normal((n_o // 64, 3))     # near every edge
    hi = lo + rng.uniform(0.05, 0.5, (n_o, 3))
    print(f"case: {n_e} edges, {n_o} boxes", flush=True)
    g = CutGPU(types.SimpleNamespace(box_lo=lo, box_hi=hi, degree=3), n_e)
    for _ in range(2):
        r = g.run(torch.as_tensor(P, device="cuda"))
        step, code = r.step.cpu().numpy(), r.code.cpu().numpy()
        want, sure = _steps(P, lo, hi)
        assert np.array_equal(step[sure], want[sure])
        assert g.qp_count() == int((step == 3).sum()) > 0
        assert np.array_equal(np.isnan(r.qp_dist2.cpu().numpy()), step != 3)
        assert np.array_equal(r.n_collide.cpu().numpy(), (code == 0).sum(0))
