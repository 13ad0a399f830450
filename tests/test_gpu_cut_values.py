"""Cut-QP values where weights tie: control points on a lattice against boxes on
the same lattice, each also given as a polytope of six rows.  The optimum is the
squared distance of conv(P) and the box either way; the box's comes from the
distance iteration (gap 1e-13), the polytope's from the value pass (gap 1e-11)."""
import types

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0.0, 1e6])
@pytest.mark.parametrize("degree", [1, 2, 3, 5, 7, 9])
def test_box_as_polytope(degree, offset):
    import torch
    from paper_2411_13507_amd.api import CutGPU
    rng = np.random.default_rng(degree)
    n, n_box = 2000, 40
    P = rng.integers(0, 7, (n, degree + 1, 3)).astype(float)
    P[:300] = P[:300, :1] + np.linspace(0, 1, degree + 1)[None, :, None] * (P[:300, -1:] - P[:300, :1])
    P[300:600, :, 2] = 3.0
    lo = rng.integers(0, 6, (n_box, 3)).astype(float)
    hi = lo + rng.integers(1, 3, (n_box, 3))
    # (multiples of 1/64: moved by an offset, every coordinate and difference stays exact)
    P, lo, hi = (v + np.array([offset, -offset, offset]) for v in (np.round(P * 64) / 64, lo, hi))
    A = np.concatenate([np.eye(3), -np.eye(3)])
    prob = types.SimpleNamespace(box_lo=lo, box_hi=hi, degree=degree, pob_off=(6 * np.arange(n_box + 1)).astype(np.int32),
                                 pob_A=np.tile(A, (n_box, 1)), pob_b=np.concatenate([hi, -lo], 1).reshape(-1))
    r = CutGPU(prob, n).run(torch.as_tensor(P, device="cuda"))
    code, step, d2 = (t.cpu().numpy() for t in (r.code, r.step, r.qp_dist2))
    free = (step[:n_box] == 3) & (step[n_box:] == 3) & (code[:n_box] == 1) & (code[n_box:] == 1)
    assert free.sum() > 100
    a, b = d2[:n_box][free], d2[n_box:][free]
    err = np.abs(a - b) / a
    print(f"case: degree {degree}, offset {offset}, {free.sum()} values, largest relative difference {err.max():.1e}", flush=True)
    assert err.max() <= 1e-9


def test_lanes_agree():
    """A pair whose dual gap lands on the stopping bound: the wavefront goes on or
    stops as one (where the lanes' sums differ in the last bit, one in twenty of
    its copies, moved by 1e-13, ends at a value near 0)."""
    import torch
    from oracle.cut import cut_qp_poly
    from paper_2411_13507_amd.api import CutGPU
    P = np.array([[0.6258225018000105, -0.8665305072438529, 7.204433177859257],
                  [0.8310452188788373, -0.4719735481173304, 0.6485768129302807],
                  [0.7483986540828451, -2.257931254962589, 4.9519576763979725],
                  [1.231659543823465, 0.03068490282195896, 8.943219434503847],
                  [1.5160104932492184, 0.8034826711387901, 4.8872908030357785],
                  [1.70266510176027, 0.22814663010662672, 2.595700930353898],
                  [2.55861944502551, -0.3037201771566187, 2.7341606191380143],
                  [1.4110871187217402, -0.6644989102349486, 4.910266135740609],
                  [2.1056270632851875, -1.2444474079033425, 3.0978571895319225],
                  [2.245857084255657, -2.826452161798948, 3.0841139542863214]])
    A = np.array([[5.1787698410098555, 5.1787698410098555, 5.1787698410098555],
                  [5.7248299060613475, -5.7248299060613475, -5.7248299060613475],
                  [-1.812954810549594, 1.812954810549594, -1.812954810549594],
                  [-0.195215212159489, -0.195215212159489, 0.195215212159489]])
    b = np.array([24.09695237082329, -12.36115908031213, -2.0267513046806, 0.19140264532757648])
    want = cut_qp_poly(P, A, b).value
    rng = np.random.default_rng(0)
    Q = np.concatenate([P[None], np.stack([P[rng.permutation(10)] for _ in range(50)]),
                        P[None] + 1e-13 * rng.standard_normal((2000, 10, 3))])
    prob = types.SimpleNamespace(box_lo=np.zeros((0, 3)), box_hi=np.zeros((0, 3)), degree=9,
                                 pob_off=np.array([0, 4], np.int32), pob_A=A, pob_b=b)
    v = CutGPU(prob, len(Q)).run(torch.as_tensor(Q, device="cuda")).qp_dist2.cpu().numpy().ravel()
    # the move changes the value by less than 2 |A| 1e-12 sqrt(value)
    assert np.abs(v - want).max() <= 1e-9 * want
