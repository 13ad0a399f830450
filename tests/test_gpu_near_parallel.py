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


def _turned_paths(b, P, paths, delta):
    """Some paths of ``b`` with the rows of every segment doubled as above."""
    import dataclasses
    seg_off, A, f, po, H, h0, G, ro, ho = [0], [], [], [0], [], [], [], [0], [0]
    for c in paths:
        ch = b.chain(c)
        for s, seg in enumerate(ch["segments"]):
            t = _turned(np.random.default_rng([c, s]), dict(seg, x0=ch["x0"]), P[int(b.seg_off[c]) + s], delta)
            A.append(t["A_face"]); f.append(t["b_face"]); po.append(po[-1] + len(f[-1]))
            H.append(t["H"].ravel()); h0.append(t["h0"]); G.append(t["G"])
            ro.append(ro[-1] + len(h0[-1])); ho.append(ho[-1] + H[-1].size)
        seg_off.append(seg_off[-1] + len(ch["segments"]))
    return dataclasses.replace(
        b, seg_off=np.asarray(seg_off, np.int64), poly_off=np.asarray(po, np.int32), A_face=np.concatenate(A),
        b_face=np.concatenate(f), poly_idx=np.arange(len(A), dtype=np.int32), reach_off=np.asarray(ro, np.int64),
        H_off=np.asarray(ho, np.int64), H=np.concatenate(H), h0=np.concatenate(h0), G=np.concatenate(G),
        x0=b.x0[paths], goal=b.goal[paths])


def _path_excess(b, c, P):
    """As _excess, over the segments of path c (control points P [segments, points, 3])."""
    ch, x0 = b.chain(c), b.x0[c, :3]
    worst = -np.inf
    for s, seg in enumerate(ch["segments"]):
        Q = P[s]
        sv, sa = b.degree / b.T, b.degree * (b.degree - 1) / b.T ** 2
        bound = seg["b_face"] - seg["A_face"] @ x0
        worst = max(worst, (((Q - x0) @ seg["A_face"].T - bound) / (1 + np.abs(bound))).max())
        worst = max(worst, (np.abs(np.diff(Q, axis=0)).max() * sv - b.vmax) / (1 + b.vmax),
                    (np.abs(np.diff(Q, 2, axis=0)).max() * sa - b.amax) / (1 + b.amax))
        H, G = seg["H"], seg["G"]
        bound = seg["h0"] - H.reshape(len(H), -1, 3).sum(1) @ x0 + G[:, :3] @ x0
        v = H @ (Q - x0).ravel()
        if s == 0:
            bound = bound + G[:, 3:] @ b.x0[c, 3:]
        else:
            v = v - G[:, :3] @ (Q[0] - x0) - G[:, 3:] @ (sv * (Q[1] - Q[0]))
        worst = max(worst, ((v - bound) / (1 + np.abs(bound))).max())
    return worst


@pytest.mark.parametrize("copies", [1, 32], ids=["one-pass", "two-pass"])
@pytest.mark.parametrize("delta", [1e-3, 3e-5, 1e-6])
def test_path_rows_hold(delta, copies):
    from tests.test_gpu_chains import _opts, gpu_chains
    from workloads import gen
    base = gen.gen_cfg3(indices=range(64))
    _, ref = gpu_chains(base, _opts(0))
    use = np.flatnonzero(ref["status"] == 0)
    b = _turned_paths(base, ref["P"].reshape(-1, 8, 3), use, delta)
    big = gen.concat_chains([b] * copies)       # (more than four paths per CU take two passes)
    for admm in (0, None):
        _, out = gpu_chains(big, _opts(admm))
        P = out["P"].reshape(-1, 8, 3)
        ok = [c for c in range(b.n) if out["status"][c] == 0]
        worst = max(_path_excess(b, c, P[b.seg_off[c]:b.seg_off[c + 1]]) for c in ok)
        print(f"case: delta {delta}, admm_iters {admm}: {len(ok)} of {b.n} solved, largest excess {worst:.1e}", flush=True)
        assert len(ok) >= 0.9 * b.n
        assert worst <= 2e-11
