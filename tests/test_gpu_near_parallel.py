"""Problems in which every face and every reachable row has a copy turned by a
small angle about the optimum (a face about the control point that comes closest
to it): warm starts propose both, the dual step drops one of them, and the working
set's factor, whose entries grow like one over the angle while both are in it, has
to be as accurate afterwards as if the pair had never met.

The bound is the solver's own contract: a row outside the working set is violated
by at most feas_tol (1e-11) times 1 + |bound|, and a row inside it holds to
rounding (some 1e3 ulps of quantities of a few units, below 1e-12)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _instances(p, n=64):
    from workloads import gen
    out = []
    for i in range(n):
        rng = np.random.default_rng([p, 5, i])
        c = rng.uniform(2, 8, 3)
        A, b, w = gen._box_polytope(rng, int(rng.integers(8, 20)), c)
        s, g = gen._sample_in(rng, A, b, c, 0.95 * w), gen._sample_in(rng, A, b, c, 0.95 * w)
        H, h0, G = gen._reach_block(rng, 24, p, 0.9, 2.6)
        out.append(dict(p=p, T=1.0, vmax=3.0, amax=5.0, A_face=A, b_face=b, H=H, h0=h0, G=G,
                        x0=np.concatenate([s, rng.uniform(-1, 1, 3)]), goal=g))
    return out


def _turned(rng, inst, P, delta):
    """``inst`` with, of each row, a copy turned by ``delta`` whose slack at the
    points P differs from the row's by up to 1e-2 ``delta``."""
    A, b, H, h0 = inst["A_face"], inst["b_face"], inst["H"], inst["h0"]

    def turn(R):
        u = rng.standard_normal(R.shape)
        u -= (u * R).sum(1, keepdims=True) / (R * R).sum(1, keepdims=True) * R
        return R + delta * u / np.linalg.norm(u, axis=1, keepdims=True) * np.linalg.norm(R, axis=1, keepdims=True)

    slack = b - P[1:-1] @ A.T                                     # [points, faces]
    k = slack.argmin(0)
    B, K = turn(A), turn(H)
    bb = (B * P[1:-1][k]).sum(1) + slack[k, np.arange(len(b))] + 1e-2 * delta * rng.uniform(-1, 1, len(b))
    kk = h0 + (K - H) @ P.ravel() + 1e-2 * delta * rng.uniform(-1, 1, len(h0))
    return dict(inst, A_face=np.concatenate([A, B]), b_face=np.concatenate([b, bb]), H=np.concatenate([H, K]),
                h0=np.concatenate([h0, kk]), G=np.concatenate([inst["G"]] * 2))


def _excess(inst, P):
    """Largest violation over 1 + |bound| of one segment's rows (bounds relative to
    the start, as the solver has them)."""
    p, T = len(P) - 1, inst["T"]
    bound = inst["b_face"] - inst["A_face"] @ P[0]
    face = ((P[1:-1] - P[0]) @ inst["A_face"].T - bound) / (1 + np.abs(bound))
    vel = np.abs(np.diff(P, axis=0)) * p / T - inst["vmax"]
    acc = np.abs(np.diff(P, 2, axis=0)) * p * (p - 1) / T ** 2 - inst["amax"]
    bound = inst["h0"] + inst["G"] @ inst["x0"] - inst["H"].reshape(len(inst["h0"]), -1, 3).sum(1) @ P[0]
    reach = (inst["H"] @ (P - P[0]).ravel() - bound) / (1 + np.abs(bound))
    return max(face.max(), vel.max() / (1 + inst["vmax"]), acc.max() / (1 + inst["amax"]), reach.max())


def _solve(insts, iters):
    import torch
    from paper_2411_13507_amd import _lib
    from paper_2411_13507_amd.api import SegmentBatchGPU
    from workloads import gen
    b = gen.from_instances(insts)
    gb = SegmentBatchGPU(b)
    o = _lib.default_opts()
    if iters is not None:
        o.admm_iters = iters
    r = gb.solve(torch.as_tensor(b.x0, device="cuda"), torch.as_tensor(b.goal, device="cuda"), opts=o)
    P = r.P.cpu().numpy().reshape(len(insts), -1, 3)
    return r.status.cpu().numpy(), P, r.cost.cpu().numpy()


@pytest.mark.parametrize("p", [3, 5, 7, 9])
@pytest.mark.parametrize("delta", [1e-4, 1e-6, 3e-8])
def test_segment_rows_hold(p, delta):
    base = _instances(p)
    st, P, _ = _solve(base, 0)
    use = np.flatnonzero(st == 0)
    assert len(use) >= 8
    insts = [_turned(np.random.default_rng([p, i]), base[i], P[i], delta) for i in use]
    for iters in (0, None, 40):
        st, Q, cost = _solve(insts, iters)
        ok = np.flatnonzero(st == 0)
        worst = max((_excess(insts[i], Q[i]) for i in ok), default=0.0)
        print(f"case: p {p}, delta {delta}, admm_iters {iters}: {len(ok)} of {len(insts)} solved, "
              f"largest excess {worst:.1e}", flush=True)
        assert len(ok) >= 0.9 * len(insts)
        assert worst <= 2e-11
