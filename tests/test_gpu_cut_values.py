"""Cut-QP values where weights tie: control points on a lattice against boxes on
the same lattice, each also given as a polytope of six rows.  The optimum is the
squared distance of conv(P) and the box either way; the box's comes from the
distance iteration (gap 1e-13), the polytope's from the value pass (gap 1e-11)."""
import types

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("degree", [1, 2, 3, 5, 7, 9])
def test_box_as_polytope(degree):
    import torch
    from paper_2411_13507_amd.api import CutGPU
    rng = np.random.default_rng(degree)
    n, n_box = 2000, 40
    P = rng.integers(0, 7, (n, degree + 1, 3)).astype(float)
    P[:300] = P[:300, :1] + np.linspace(0, 1, degree + 1)[None, :, None] * (P[:300, -1:] - P[:300, :1])
    P[300:600, :, 2] = 3.0
    lo = rng.integers(0, 6, (n_box, 3)).astype(float)
    hi = lo + rng.integers(1, 3, (n_box, 3))
    A = np.concatenate([np.eye(3), -np.eye(3)])
    prob = types.SimpleNamespace(box_lo=lo, box_hi=hi, degree=degree, pob_off=(6 * np.arange(n_box + 1)).astype(np.int32),
                                 pob_A=np.tile(A, (n_box, 1)), pob_b=np.concatenate([hi, -lo], 1).reshape(-1))
    r = CutGPU(prob, n).run(torch.as_tensor(P, device="cuda"))
    code, step, d2 = (t.cpu().numpy() for t in (r.code, r.step, r.qp_dist2))
    free = (step[:n_box] == 3) & (step[n_box:] == 3) & (code[:n_box] == 1) & (code[n_box:] == 1)
    assert free.sum() > 100
    a, b = d2[:n_box][free], d2[n_box:][free]
    err = np.abs(a - b) / a
    print(f"case: degree {degree}, {free.sum()} values, largest relative difference {err.max():.1e}", flush=True)
    assert err.max() <= 1e-9
