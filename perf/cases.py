"""The work that a user of the Bezier-graph library has it do, as cases that can
be timed: one dict of plain values per case, prepared on the GPU from a seed and
run through the public entry points.

Six kinds of work, in the order a planner meets them:

* ``graph``    which nodes are joined (reachability test of every ordered pair);
* ``planes``   nearest obstacle and separating plane of every node;
* ``cut``      graph edges against boxes and convex polytopes;
* ``segments`` one QP per candidate edge, and its derivatives;
* ``paths``    one QP per multi-segment path;
* ``mpc``      refinement of a path over a horizon.

The distributions are those of the repository's workloads (a 10 m cube, a few
hundred box obstacles, free-space polytopes with 8-24 faces, 32 reachable rows
per edge, horizons of 50 steps of 0.1 s), drawn here with torch on the GPU so
that preparing a case is quick.

Residuals and step counts describe how a solver got to its result and not the
result, so ``run`` does not return them.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2411_13507_amd import _lib, torch_fn
from paper_2411_13507_amd.api import (ChainBatchGPU, CutGPU, GraphGPU, MpcGPU, MpcResult, SegmentBatchGPU,
                                      adjacent_hyperplanes)

F64 = torch.float64
DEV = "cuda"
VMAX, AMAX, T_SEG = 3.0, 5.0, 1.0


# --------------------------------------------------------------------------
# cases
# --------------------------------------------------------------------------

def _segments(name, n, degree=(7, 7), reach=(32, 32), faces=(8, 24), solver="polish", use="solve_backward",
              shared=False, pinned=False):
    return dict(name=name, kind="segments", n=n, p_lo=degree[0], p_hi=degree[1], r_lo=reach[0], r_hi=reach[1],
                f_lo=faces[0], f_hi=faces[1], solver=solver, use=use, shared=shared, pinned=pinned)


def listed():
    return [
        # a few edges inside a training or trajectory-optimisation loop: autograd
        # with the default options, where latency and launches count
        _segments("edges64_autograd_default", 64, faces=(6, 6), solver="default", use="autograd"),
        # the edges of one replanning query with the options left at their defaults
        # (FP32 warm start, then the FP64 polish), and their derivatives
        _segments("edges4k_default", 4096, solver="default"),
        # a whole graph's edges with the tuned options (polish only): forward and
        # backward, the throughput case
        _segments("edges50k_polish", 50_000),
        # one reachable block for all edges and a pinned start velocity (a robot
        # with one set of dynamics, starting from its full state)
        _segments("edges12k_shared_pinned", 12_345, shared=True, pinned=True),
        # mixed degrees, 6-40 faces, 16-128 rows: a graph whose edges differ, forward only
        _segments("edges30k_uneven", 30_000, degree=(3, 9), reach=(16, 128), faces=(6, 40), use="solve"),
        # candidate paths of 4-12 joined segments
        dict(name="paths1024", kind="paths", n=1024, s_lo=4, s_hi=12, solver="polish"),
        # the graph of 5,000 nodes (the planner's own size)
        dict(name="graph5000_m64", kind="graph", n=5000, m=64, zorder=True),
        # separating planes of the same nodes
        dict(name="planes5000_b200", kind="planes", n=5000, boxes=200),
        # an environment update: 50,000 edges against boxes, codes and counts only
        dict(name="cut50k_b200", kind="cut", nodes=5000, boxes=200, polys=0, degree=7, values=False),
        # boxes and convex polytopes, with the deciding steps and the Cut-QP values
        # (the call's defaults)
        dict(name="cut20k_b200_p100_values", kind="cut", nodes=2000, boxes=200, polys=100, degree=7, values=True),
        # refinement of one robot's few candidate paths: latency
        dict(name="mpc16_n50", kind="mpc", n=16, N=50, extra=4),
        # a large batch of horizons
        dict(name="mpc4096_n50", kind="mpc", n=4096, N=50, extra=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["segments"] * 5 + ["paths", "graph", "planes"] + ["cut"] * 2 + ["mpc"] * 2)
    if kind == "segments":
        uneven = rng.random() < 0.3
        c = _segments("", _log_int(rng, 16, 30_000 if uneven else 50_000))
        if uneven:
            c.update(p_lo=3, p_hi=rng.randint(5, 9), r_lo=rng.randint(0, 16), r_hi=rng.randint(32, 128),
                     f_lo=6, f_hi=rng.randint(12, 40))
        else:
            p, r = rng.randint(3, 9), rng.randint(8, 100)
            c.update(p_lo=p, p_hi=p, r_lo=r, r_hi=r, f_hi=rng.randint(8, 40))
        c["n"] = max(16, min(c["n"], int(50_000 * 3e4 / ((c["p_hi"] + 1) ** 2 * (c["r_hi"] + 40) * 6.5))))
        c["solver"] = rng.choice(["polish", "polish", "default"])
        if c["solver"] == "default":
            c["n"] = min(c["n"], 12_000)
        c["use"] = rng.choice(["solve", "solve_backward", "autograd"])
        c["shared"] = not uneven and rng.random() < 0.25
        c["pinned"] = rng.random() < 0.25
    elif kind == "paths":
        lo = rng.randint(1, 8)
        c = dict(kind=kind, n=_log_int(rng, 16, 1024), s_lo=lo, s_hi=rng.randint(lo, 12),
                 solver=rng.choice(["polish", "polish", "default"]))
        if c["solver"] == "default":
            c["n"] = min(c["n"], 400)
    elif kind == "graph":
        c = dict(kind=kind, n=_log_int(rng, 200, 8000), m=rng.randint(8, 128), zorder=rng.random() < 0.75)
    elif kind == "planes":
        c = dict(kind=kind, n=_log_int(rng, 50, 50_000), boxes=_log_int(rng, 10, 500))
    elif kind == "cut":
        c = dict(kind=kind, nodes=_log_int(rng, 50, 5000), boxes=_log_int(rng, 10, 300),
                 polys=rng.choice([0, rng.randint(1, 100)]), degree=rng.choice([3, 5, 7, 7, 9]),
                 values=rng.random() < 0.5)
    else:
        c = dict(kind=kind, n=_log_int(rng, 1, 4096), N=rng.randint(8, 60), extra=rng.randint(0, 16))
        c["n"] = max(1, min(c["n"], int(4096 * 50 * 16 / (c["N"] * (12 + c["extra"])))))
    c.pop("name", None)
    return c


# --------------------------------------------------------------------------
# inputs (torch on the GPU, from the seed alone)
# --------------------------------------------------------------------------

class _Rand:
    """Draws from ``seed``; whole numbers that fix the sizes of the outputs (degrees,
    rows, faces, segments, polytope of an edge) come from a stream of their own, so
    that a case has the same shapes for every seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV).manual_seed(int(seed) % (1 << 62))
        self.sizes = torch.Generator(device=DEV).manual_seed(2411)

    def uniform(self, lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(shape, dtype=F64, device=DEV, generator=self.g)

    def normal(self, *shape):
        return torch.randn(shape, dtype=F64, device=DEV, generator=self.g)

    def integers(self, lo, hi, *shape):   # hi included
        return torch.randint(lo, hi + 1, shape, device=DEV, generator=self.sizes)

    def unit(self, *shape):
        v = self.normal(*shape)
        return v / v.norm(dim=-1, keepdim=True)


def _boxes(R, n):
    c, s = R.uniform(0.0, 10.0, n, 3), R.uniform(0.2, 1.5, n, 3)
    return c - s / 2, c + s / 2


def _outside(R, n, lo, hi, reject=None):
    """n points of the cube outside every box (and outside ``reject``)."""
    got, have = [], 0
    while have < n:
        x = R.uniform(0.0, 10.0, 2 * n + 64, 3)
        hit = torch.zeros(len(x), dtype=torch.bool, device=DEV)
        for a in range(0, len(lo), 64):
            hit |= ((x[:, None] >= lo[a:a + 64]) & (x[:, None] <= hi[a:a + 64])).all(-1).any(-1)
        if reject is not None:
            hit |= reject(x)
        x = x[~hit]
        got.append(x)
        have += len(x)
    return torch.cat(got)[:n]


def _polytopes(R, centres, nf, fmax):
    """A bounded polytope of nf[i] faces round every centre: six axis faces at
    half-widths U[0.5, 2] and Gaussian cuts at U[0.5, 2], padded to fmax rows
    (0.x <= 1)."""
    n = len(centres)
    w = R.uniform(0.5, 2.0, n, 3)
    A = torch.zeros(n, fmax, 3, dtype=F64, device=DEV)
    A[:, :3], A[:, 3:6] = torch.eye(3, dtype=F64, device=DEV), -torch.eye(3, dtype=F64, device=DEV)
    A[:, 6:] = R.unit(n, max(0, fmax - 6), 3)
    b = torch.ones(n, fmax, dtype=F64, device=DEV)
    b[:, :3], b[:, 3:6] = centres + w, -(centres - w)
    b[:, 6:] = (A[:, 6:] * centres[:, None]).sum(-1) + R.uniform(0.5, 2.0, n, max(0, fmax - 6))
    pad = torch.arange(fmax, device=DEV) >= nf[:, None]
    A[pad], b[pad] = 0.0, 1.0
    return A, b, w


def _inside(A, b, x):
    """x [n, k, 3] in the polytopes A [n, f, 3], b [n, f]: [n, k]."""
    ok = torch.ones(x.shape[:2], dtype=torch.bool, device=DEV)
    for f in range(A.shape[1]):
        ok &= (x * A[:, f, None]).sum(-1) <= b[:, f, None]
    return ok


def _first(x, ok, fallback):
    """The first accepted of the candidates x [n, k, 3], else the fallback."""
    k = ok.to(torch.int8).argmax(1)
    return torch.where(ok.any(1)[:, None], x[torch.arange(len(x), device=DEV), k], fallback), ok.any(1)


def _sample_in(R, A, b, c, w, k=64):
    x = c[:, None] + w[:, None] * R.uniform(-1.0, 1.0, len(c), k, 3)
    return _first(x, _inside(A, b, x), c)[0]


def _offsets(counts, dtype):
    return torch.cat([torch.zeros(1, dtype=torch.int64, device=DEV), counts.cumsum(0)]).to(dtype)


def _flat(A, b, nf):
    keep = torch.arange(A.shape[1], device=DEV) < nf[:, None]
    return _offsets(nf, torch.int32), A[keep], b[keep]


def _reach(R, p, r, h0):
    """Reachable rows of blocks with degree p[i] and r[i] rows: unit Gaussian rows,
    right-hand sides U[h0], G = N(0, 0.1^2) plus the part that follows the start."""
    ncol = 3 * (p + 1)
    reach_off, H_off = _offsets(r, torch.int64), _offsets(r * ncol, torch.int64)
    total = int(reach_off[-1])
    H = torch.empty(int(H_off[-1]), dtype=F64, device=DEV)
    G = 0.1 * R.normal(total, 6)
    blk = torch.repeat_interleave(torch.arange(len(p), device=DEV), r)
    local = torch.arange(total, device=DEV) - reach_off[blk]
    start = H_off[blk] + local * ncol[blk]
    for d in torch.unique(p).tolist():
        rows = torch.nonzero(p[blk] == d)[:, 0]
        h = R.unit(len(rows), 3 * (d + 1))
        H[(start[rows][:, None] + torch.arange(3 * (d + 1), device=DEV)).reshape(-1)] = h.reshape(-1)
        G[rows, :3] += h.reshape(len(rows), d + 1, 3).sum(1)
    return reach_off, H_off, H, R.uniform(h0[0], h0[1], total), G


def _segment_inputs(case, seed):
    R, n = _Rand(seed), case["n"]
    lo, hi = _boxes(R, 200)
    n_poly = min(2000, max(50, n))
    c = _outside(R, n_poly, lo, hi)
    nf = R.integers(case["f_lo"], case["f_hi"], n_poly)
    A, b, w = _polytopes(R, c, nf, case["f_hi"])
    near = torch.cdist(c, c).fill_diagonal_(float("inf")).topk(4, largest=False).indices
    j = R.integers(0, n_poly - 1, n)
    start = torch.empty(n, 3, dtype=F64, device=DEV)
    goal = torch.empty(n, 3, dtype=F64, device=DEV)
    for s in range(0, n, 8192):
        k = j[s:s + 8192]
        Aj, bj, cj, wj = A[k], b[k], c[k], w[k]
        start[s:s + 8192] = _sample_in(R, Aj, bj, cj, wj)
        x = cj[:, None] + wj[:, None] * R.uniform(-1.0, 1.0, len(k), 128, 3)
        own = _inside(Aj, bj, x)
        g, found = _first(x, own, cj)
        found = torch.zeros_like(found)
        order = torch.rand(len(k), 4, device=DEV, generator=R.g).argsort(1)
        for t in range(4):
            nb = near[k].gather(1, order[:, t:t + 1])[:, 0]
            gt, ft = _first(x, own & _inside(A[nb], b[nb], x), cj)
            g = torch.where((ft & ~found)[:, None], gt, g)
            found |= ft
        goal[s:s + 8192] = g
    x0 = torch.cat([start, R.uniform(-1.0, 1.0, n, 3)], 1)
    p = R.integers(case["p_lo"], case["p_hi"], n)
    r = R.integers(case["r_lo"], case["r_hi"], n)
    q = SimpleNamespace(degree=p, T=torch.full((n,), T_SEG, dtype=F64), vmax=VMAX, amax=AMAX, poly_idx=j,
                        pin_v0=case["pinned"], reach_idx=None)
    q.poly_off, q.A_face, q.b_face = _flat(A, b, nf)
    if case["shared"]:
        q.reach_idx = torch.zeros(n, dtype=torch.int32)
        q.reach_off, q.H_off, q.H, q.h0, q.G = _reach(R, p[:1], r[:1], (1.6, 3.6))
    else:
        q.reach_off, q.H_off, q.H, q.h0, q.G = _reach(R, p, r, (1.3, 3.3))
    return _host(q), x0.contiguous(), goal, R


def _path_inputs(case, seed):
    R, n, F = _Rand(seed), case["n"], 24
    S = R.integers(case["s_lo"], case["s_hi"], n)
    nf = R.integers(8, F, n, case["s_hi"])
    c = R.uniform(2.0, 8.0, n, 3)
    A, b, w = _polytopes(R, c, nf[:, 0], F)
    walk = [(A, b, c, w)]
    for s in range(1, case["s_hi"]):
        A0, b0, c0, w0 = walk[-1]
        new = tuple(torch.empty_like(t) for t in walk[-1])
        todo = torch.arange(n, device=DEV)
        for _ in range(50):
            ck = c0[todo] + R.unit(len(todo), 3) * R.uniform(0.8, 1.5, len(todo), 1)
            Ak, bk, wk = _polytopes(R, ck, nf[todo, s], F)
            x = c0[todo][:, None] + w0[todo][:, None] * R.uniform(-1.0, 1.0, len(todo), 256, 3)
            ok = (_inside(A0[todo], b0[todo], x) & _inside(Ak, bk, x)).any(1)
            for t, v in zip(new, (Ak, bk, ck, wk)):
                t[todo[ok]] = v[ok]
            todo = todo[~ok]
            if not len(todo):
                break
        assert not len(todo), "no overlapping polytope found"
        walk.append(new)
    last = S - 1
    at = torch.arange(n, device=DEV)
    tab = [torch.stack(v, 1) for v in zip(*walk)]          # [n, s_hi, ...]
    start = _sample_in(R, walk[0][0], walk[0][1], walk[0][2], walk[0][3])
    goal = _sample_in(R, tab[0][at, last], tab[1][at, last], tab[2][at, last], tab[3][at, last])
    live = torch.arange(case["s_hi"], device=DEV) < S[:, None]
    q = SimpleNamespace(seg_off=_offsets(S, torch.int64), degree=7, T=T_SEG, vmax=VMAX, amax=AMAX)
    q.poly_off, q.A_face, q.b_face = _flat(tab[0][live], tab[1][live], nf[live])
    n_seg = int(S.sum())
    q.poly_idx = torch.arange(n_seg)
    full = lambda v: torch.full((n_seg,), v, dtype=torch.int64, device=DEV)  # noqa: E731
    q.reach_off, q.H_off, q.H, q.h0, q.G = _reach(R, full(7), full(32), (2.0, 4.0))
    x0 = torch.cat([start, R.uniform(-1.0, 1.0, n, 3)], 1)
    return _host(q), x0.contiguous(), goal


def _graph_inputs(case, seed):
    R, n, m = _Rand(seed), case["n"], case["m"]
    V = R.uniform(0.0, 10.0, n, 3)
    if case["zorder"]:   # nodes numbered along a space-filling curve
        cell = (V / 10.0 * 1024).long().clamp_(0, 1023)
        code = torch.zeros(n, dtype=torch.int64, device=DEV)
        for bit in range(10):
            for k in range(3):
                code |= ((cell[:, k] >> bit) & 1) << (3 * bit + k)
        V = V[code.argsort()].contiguous()
    a = R.unit(m, 3)
    return _host(SimpleNamespace(F1=-a, F2=a + 0.02 * R.normal(m, 3), G=R.uniform(0.85, 1.1, m))), V


def _cut_inputs(case, seed):
    R, n, p = _Rand(seed), case["nodes"], case["degree"]
    lo, hi = _boxes(R, case["boxes"])
    np_ = case["polys"]
    c, w = R.uniform(0.0, 10.0, np_, 3), R.uniform(0.1, 0.75, np_, 3)
    k = R.integers(2, 10, np_)
    I3 = torch.eye(3, dtype=F64, device=DEV).expand(np_, 3, 3)
    cuts = R.unit(np_, 10, 3)
    A = torch.cat([I3, -I3, cuts], 1)
    b = torch.cat([c + w, -(c - w), (cuts * c[:, None]).sum(-1) + R.uniform(0.1, 0.75, np_, 10)], 1)
    pad = torch.arange(16, device=DEV) >= (6 + k)[:, None]
    Ap, bp = A.masked_fill(pad[..., None], 0.0), b.masked_fill(pad, 1.0)

    def in_poly(x):
        hit = torch.zeros(len(x), dtype=torch.bool, device=DEV)
        for i in range(np_):
            hit |= ((x[:, None] * Ap[i]).sum(-1) <= bp[i]).all(-1)
        return hit

    V = _outside(R, n, lo, hi, in_poly if np_ else None)
    nbr = torch.cdist(V, V).fill_diagonal_(float("inf")).topk(10, largest=False).indices
    a, z = V.repeat_interleave(10, 0), V[nbr.reshape(-1)]
    t = torch.arange(p + 1, dtype=F64, device=DEV) / p
    P = a[:, None] + t[None, :, None] * (z - a)[:, None]
    P[:, 1:p] += R.normal(len(a), p - 1, 3) * (0.15 * (z - a).norm(dim=1))[:, None, None]
    off, Af, bf = _flat(A, b, 6 + k)
    q = SimpleNamespace(box_lo=lo, box_hi=hi, degree=p, pob_off=off, pob_A=Af, pob_b=bf)
    return _host(q), P.contiguous()


def _mpc_inputs(case, seed):
    R, n, N, dt = _Rand(seed), case["n"], case["N"], 0.1
    e = torch.eye(3, dtype=F64, device=DEV)
    O, Z = torch.zeros(3, 3, dtype=F64, device=DEV), torch.zeros(6, 6, dtype=F64, device=DEV)
    dirs = R.unit(case["extra"], 3)
    z3 = torch.zeros(case["extra"], 3, dtype=F64, device=DEV)
    sgn = torch.cat([e, -e])
    F1 = torch.cat([Z, torch.cat([torch.cat([O, O]), -sgn], 1), torch.cat([z3, -dirs], 1)])
    F2 = torch.cat([torch.cat([torch.cat([O, O]), sgn], 1)] * 2 + [torch.cat([z3, dirs], 1)])
    G = torch.cat([torch.full((6,), 2.0, dtype=F64, device=DEV), torch.full((6,), 4.0 * dt, dtype=F64, device=DEV),
                   R.uniform(0.05, 0.09, case["extra"])])
    amp, om, ph = R.uniform(0.2, 0.5, 2, n, 1, 3), R.uniform(1.5, 3.0, 2, n, 1, 3), R.uniform(0, 2 * math.pi, 2, n, 1, 3)
    t = dt * torch.arange(N + 1, dtype=F64, device=DEV)[:, None]
    v0, p0 = R.uniform(-0.5, 0.5, n, 1, 3), R.uniform(2.0, 8.0, n, 1, 3)
    vel = v0 + (amp / om * (ph.cos() - (om * t + ph).cos())).sum(0)
    pos = p0 + v0 * t + (amp / om * (t * ph.cos() - ((om * t + ph).sin() - ph.sin()) / om)).sum(0)
    ref = torch.cat([pos, vel], 2)
    acc, v = (amp * (om * t + ph).sin()).sum(0)[:, :N], vel[:, :N]
    side = acc - (acc * v).sum(-1, keepdim=True) / (v * v).sum(-1, keepdim=True).clamp_min(1e-12) * v
    nrm = -side / side.norm(dim=-1, keepdim=True).clamp_min(1e-12) + 0.3 * R.normal(n, N, 3)
    nrm = nrm / nrm.norm(dim=-1, keepdim=True)
    gap = R.uniform(0.05, 0.25, n, N)
    gap[:, 0] = R.uniform(0.22, 0.5, n)
    planes = torch.cat([nrm, ((nrm * pos[:, :N]).sum(-1) - gap)[..., None]], 2)
    x0 = ref[:, 0] + torch.cat([R.uniform(-0.05, 0.05, n, 3), R.uniform(-0.1, 0.1, n, 3)], 1)
    q = SimpleNamespace(N=N, dt=dt, Q=np.diag([1.0, 1.0, 1.0, 0.1, 0.1, 0.1]), R=0.01 * np.eye(3), w=50.0,
                        F1=F1, F2=F2, G=G)
    return _host(q), x0.contiguous(), ref.contiguous(), planes.contiguous()


def _host(q):
    """The description as a program holds it before it builds a batch: numpy arrays."""
    for k, v in vars(q).items():
        if isinstance(v, torch.Tensor):
            setattr(q, k, v.cpu().numpy())
    return q


def _opts(case, store):
    o = _lib.default_opts()
    if case["solver"] == "polish":
        o.admm_iters = 0
        if case["kind"] == "segments" and case["p_hi"] > case["p_lo"]:
            o.launch_shape = 1   # what the autotuner picks for mixed degrees
    o.store_for_backward = 1 if store else 0
    return o


# --------------------------------------------------------------------------
# prepare and run
# --------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    if kind == "segments":
        q, x0, goal, R = _segment_inputs(case, seed)
        batch = SegmentBatchGPU(q, device=DEV)
        s = dict(case=case, batch=batch, x0=x0, goal=goal, opts=_opts(case, case["use"] != "solve"))
        if case["use"] != "solve":
            s["gP"], s["gf"] = R.normal(3 * batch.points_total), torch.ones(batch.N, dtype=F64, device=DEV)
        if case["use"] == "autograd":
            s["b"] = batch.b_face.clone().requires_grad_()
            s["x0"], s["goal"] = x0.requires_grad_(), goal.requires_grad_()
        else:
            s["out"] = batch.alloc_outputs()
        return s
    if kind == "paths":
        q, x0, goal = _path_inputs(case, seed)
        return dict(case=case, batch=ChainBatchGPU(q, device=DEV), x0=x0, goal=goal, opts=_opts(case, False))
    if kind == "graph":
        q, V = _graph_inputs(case, seed)
        return dict(case=case, graph=GraphGPU(q, case["n"], device=DEV), V=V)
    if kind == "planes":
        R = _Rand(seed)
        lo, hi = _boxes(R, case["boxes"])
        return dict(case=case, X=R.uniform(0.0, 10.0, case["n"], 3), lo=lo.contiguous(), hi=hi.contiguous())
    if kind == "cut":
        q, P = _cut_inputs(case, seed)
        cut = CutGPU(q, len(P), device=DEV)
        return dict(case=case, cut=cut, P=P, out=cut.alloc())
    q, x0, ref, planes = _mpc_inputs(case, seed)
    mpc = MpcGPU(q, case["n"], device=DEV)
    return dict(case=case, mpc=mpc, x0=x0, ref=ref, planes=planes, out=mpc.alloc())


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "segments":
        batch = state["batch"]
        if case["use"] == "autograd":
            P, f, status = torch_fn.solve(state["x0"], state["goal"], state["b"], batch, state["opts"])
            gx, gg, gb = torch.autograd.grad((P, f), (state["x0"], state["goal"], state["b"]),
                                             (state["gP"], state["gf"]))
            return dict(P=P, cost=f, status=status, grad_x0=gx, grad_goal=gg, grad_b=gb)
        r = batch.solve(state["x0"], state["goal"], opts=state["opts"], out=state["out"])
        res = dict(P=r.P, cost=r.cost, status=r.status)
        if case["use"] == "solve_backward":
            g = batch.backward(state["gP"], state["gf"])
            res.update(grad_x0=g.x0, grad_goal=g.goal, grad_b=g.b_inst, flags=g.flags)
        return res
    if kind == "paths":
        r = state["batch"].solve(state["x0"], state["goal"], opts=state["opts"])
        return dict(P=r.P, cost=r.cost, status=r.status)
    if kind == "graph":
        adj, deg = state["graph"].run(state["V"])
        return dict(adj=adj, degree=deg)
    if kind == "planes":
        idx, point, plane = adjacent_hyperplanes(state["X"], state["lo"], state["hi"])
        return dict(index=idx, point=point, plane=plane)
    if kind == "cut":
        v = case["values"]
        r = state["cut"].run(state["P"], out=state["out"], with_step=v, with_dist=v)
        return dict(code=r.code, n_collide=r.n_collide, step=r.step if v else None, value=r.qp_dist2 if v else None)
    r: MpcResult = state["mpc"].solve(state["x0"], state["ref"], state["planes"], out=state["out"])
    return dict(X=r.X, U=r.U, cost=r.cost, status=r.status)


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------

def work(case):
    """Every input read once and every output written once; one evaluation of every
    row at the result and, for the QPs, one factorisation of the reduced Hessian."""
    kind = case["kind"]
    if kind == "segments":
        n, p, r = case["n"], (case["p_lo"] + case["p_hi"]) / 2, (case["r_lo"] + case["r_hi"]) / 2
        f, nv = (case["f_lo"] + case["f_hi"]) / 2, 3 * ((case["p_lo"] + case["p_hi"]) / 2 - 1)
        blocks = 1 if case["shared"] else n
        table = min(2000, max(50, n)) * f * 32
        by = blocks * r * (3 * (p + 1) * 8 + 56) + table + n * (72 + 12 + 24 * (p + 1) + 12)
        fl = n * (2 * nv * (2 * f + r + 5) + nv ** 3 / 3)
        if case["use"] != "solve":
            by += n * (24 * (p + 1) + 8 + 72 + 8 * f + 4)
            fl += n * 4 * nv * nv
        return dict(bytes=by, flops=fl)
    if kind == "paths":
        S = (case["s_lo"] + case["s_hi"]) / 2
        seg = case["n"] * S
        return dict(bytes=seg * (32 * (192 + 56) + 16 * 32 + 192) + case["n"] * 84,
                    flops=seg * (2 * 24 * 32 + 2 * 3 * 8 * 16 + 2 * 24 * 5) + case["n"] * 2 * 3 * (5 * S + 1) * 64)
    if kind == "graph":
        n, m = case["n"], case["m"]
        return dict(bytes=n * 24 + m * 56 + n * ((n + 31) // 32) * 4 + n * 4, flops=12 * n * m + 2 * n * n)
    if kind == "planes":
        n, b = case["n"], case["boxes"]
        return dict(bytes=n * 84 + b * 48, flops=n * b * 11)
    if kind == "cut":
        E, p = case["nodes"] * 10, case["degree"]
        pairs = E * (case["boxes"] + case["polys"])
        return dict(bytes=E * (p + 1) * 24 + pairs * (10 if case["values"] else 1) + E * 4, flops=pairs * 12)
    n, N, m = case["n"], case["N"], 12 + case["extra"]
    return dict(bytes=n * ((N + 1) * 96 + N * 56 + 60), flops=n * N * (2 * 9 * (m + 4) + 600))


# --------------------------------------------------------------------------
# the same results with plain torch in 64 bits
# --------------------------------------------------------------------------

def _ipm(H, g, A, b, iters=60):
    """Batched min 1/2 x'Hx + g'x, A x <= b (H [n,d,d] or [d,d], rows of norm 0
    are ignored): predictor-corrector interior point, then the equality-constrained
    optimum on the active rows.  Returns x, the rows taken as active (d indices and
    a mask) and whether it converged."""
    n, m, d = A.shape
    H = H.expand(n, d, d)
    nrm = A.norm(dim=-1)
    off = nrm < 1e-12
    A = A / torch.where(off, torch.ones_like(nrm), nrm)[..., None]
    dead = (off & (b < 0)).any(1)
    b = torch.where(off, torch.ones_like(b), b / torch.where(off, torch.ones_like(nrm), nrm))
    x = -torch.linalg.solve(H, g[..., None])[..., 0]
    Ax = lambda v: (A @ v[..., None])[..., 0]  # noqa: E731
    At = A.transpose(1, 2).contiguous()
    Atv = lambda v: (At @ v[..., None])[..., 0]  # noqa: E731
    s = (b - Ax(x)).clamp_min(1.0)
    lam = torch.ones_like(s)
    for _ in range(iters):
        rd, rp = (H @ x[..., None])[..., 0] + g + Atv(lam), Ax(x) + s - b
        mu = (s * lam).mean(1)
        w = lam / s
        L = torch.linalg.cholesky_ex(H + At @ (w[..., None] * A))[0]

        def step(rc):
            rhs = -rd - Atv(w * rp - rc / s)
            dx = torch.cholesky_solve(rhs[..., None], L)[..., 0]
            ds = -rp - Ax(dx)
            return dx, ds, (-rc - lam * ds) / s

        def length(v, dv):
            return torch.where(dv < 0, -v / dv, torch.full_like(v, 1e9)).amin(1).clamp(max=1.0)

        _, ds, dl = step(s * lam)
        a, c = length(s, ds), length(lam, dl)
        mua = ((s + a[:, None] * ds) * (lam + c[:, None] * dl)).mean(1)
        sig = (mua / mu).clamp(0, 1) ** 3
        dx, ds, dl = step(s * lam + ds * dl - (sig * mu)[:, None])
        a, c = 0.995 * length(s, ds), 0.995 * length(lam, dl)
        ok = torch.isfinite(dx).all(1) & (mu > 1e-14)
        a, c = torch.where(ok, a, 0.0)[:, None], torch.where(ok, c, 0.0)[:, None]
        z = lambda v: torch.nan_to_num(v)  # noqa: E731
        x, s, lam = x + a * z(dx), s + a * z(ds), lam + c * z(dl)
    k = min(d, m)
    scale = 1.0 + g.abs().amax(1)
    res = ((H @ x[..., None])[..., 0] + g + Atv(lam)).abs().amax(1)
    conv = ((Ax(x) - b).amax(1) < 1e-6) & (res < 1e-5 * scale) & ~dead   # not so where nothing is feasible
    top = torch.where(lam > s, lam, torch.full_like(lam, -1.0)).topk(k, dim=1)
    return x, top.indices, top.values > 0, conv


def _kkt(H, g, A, b, act, live, eps=0.0):
    """The optimum with the given active rows as equations (differentiable)."""
    n, _, d = A.shape
    k = act.shape[1]
    C = torch.gather(A, 1, act[..., None].expand(n, k, d)) * live[..., None]
    e = torch.gather(b, 1, act) * live
    # a row that is not taken stands as -1 on the diagonal; a taken one has -eps
    # there, which decides between rows that say the same
    K = torch.cat([torch.cat([H.expand(n, d, d), C.transpose(1, 2)], 2),
                   torch.cat([C, -torch.diag_embed(torch.where(live, eps, 1.0).to(F64))], 2)], 1)
    return torch.linalg.solve_ex(K, torch.cat([-g, e], 1)[..., None])[0][:, :d, 0]


def _bernstein_cost(p):
    """Q with cost = sum over coordinates of P_c' Q P_c = int_0^1 |b''|^2."""
    D = np.zeros((p - 1, p + 1))
    for i in range(p - 1):
        D[i, i:i + 3] = (1.0, -2.0, 1.0)
    q = p - 2
    M = np.array([[math.comb(q, i) * math.comb(q, j) / ((2 * q + 1) * math.comb(2 * q, i + j))
                   for j in range(q + 1)] for i in range(q + 1)])
    return torch.as_tensor((p * (p - 1)) ** 2 * D.T @ M @ D, dtype=F64, device=DEV)


def _derivative_rows(p):
    V, W = np.zeros((p, p + 1)), np.zeros((p - 1, p + 1))
    for i in range(p):
        V[i, i:i + 2] = (-p, p)
    for i in range(p - 1):
        W[i, i:i + 3] = p * (p - 1) * np.array((1.0, -2.0, 1.0))
    return V, W


def _kron3(M):
    return torch.as_tensor(np.kron(M, np.eye(3)), dtype=F64, device=DEV)


def _exact_segments(case, seed):
    q, x0, goal, R = _segment_inputs(case, seed)
    n = case["n"]
    deg = torch.as_tensor(q.degree, device=DEV)
    pts = int((deg + 1).sum())
    gP = R.normal(3 * pts) if case["use"] != "solve" else None
    pt = _offsets(deg + 1, torch.int64)
    po = torch.as_tensor(q.poly_off, dtype=torch.int64, device=DEV)
    pi = torch.as_tensor(q.poly_idx, dtype=torch.int64, device=DEV)
    nf = (po[1:] - po[:-1])[pi]
    fo = _offsets(nf, torch.int64)
    Af, bf = torch.as_tensor(q.A_face, device=DEV), torch.as_tensor(q.b_face, device=DEV)
    ro, ho = torch.as_tensor(q.reach_off, device=DEV), torch.as_tensor(q.H_off, device=DEV)
    Hh, h0, G = (torch.as_tensor(v, device=DEV) for v in (q.H, q.h0, q.G))
    blk = torch.arange(n, device=DEV) if q.reach_idx is None else torch.as_tensor(q.reach_idx, dtype=torch.int64, device=DEV)
    P = torch.full((3 * pts,), float("nan"), dtype=F64, device=DEV)
    cost = torch.full((n,), float("inf"), dtype=F64, device=DEV)
    gx, gg = torch.zeros(n, 6, dtype=F64, device=DEV), torch.zeros(n, 3, dtype=F64, device=DEV)
    gb = torch.zeros(int(fo[-1]), dtype=F64, device=DEV)
    fcap, rcap = int(nf.max()), int((ro[1:] - ro[:-1]).max())
    for p in torch.unique(deg).tolist():
        V, W = _derivative_rows(p)
        D = _kron3(np.concatenate([V, -V, W, -W]))
        Q3 = torch.kron(_bernstein_cost(p), torch.eye(3, dtype=F64, device=DEV))
        free = slice(6, 3 * p) if case["pinned"] else slice(3, 3 * p)
        ids = torch.nonzero(deg == p)[:, 0]
        for i in torch.split(ids, 4096):
            k = len(i)
            X, Z = x0[i].detach().requires_grad_(), goal[i].detach().requires_grad_()
            j = torch.arange(fcap, device=DEV)
            on = j < nf[i][:, None]
            at = (po[pi[i]][:, None] + j).clamp_max(len(bf) - 1)
            Bf = (bf[at] * on).detach().requires_grad_()
            An = Af[at] * on[..., None]
            l = torch.arange(rcap, device=DEV)
            r_on = l < (ro[blk[i] + 1] - ro[blk[i]])[:, None]
            ra = (ro[blk[i]][:, None] + l).clamp(max=max(len(h0) - 1, 0))
            ha = (ho[blk[i]][:, None, None] + (l[:, None] * 3 * (p + 1) + torch.arange(3 * (p + 1), device=DEV))).clamp_max(max(len(Hh) - 1, 0))
            Hr = Hh[ha] * r_on[..., None]
            hr = torch.where(r_on, h0[ra] + (G[ra] * X[:, None]).sum(-1), 1.0)
            # the pinned coordinates, in the frame of the whole control polygon
            pin = [X[:, :3]] + ([X[:, :3] + X[:, 3:] / p] if case["pinned"] else [])
            y0 = torch.cat(pin + [torch.zeros(k, free.stop - free.start, dtype=F64, device=DEV), Z], 1)
            Frow = torch.zeros(k, p + 1, fcap, p + 1, 3, dtype=F64, device=DEV)
            for s in range(p + 1):
                Frow[:, s, :, s] = An
            A = torch.cat([Frow.reshape(k, -1, 3 * (p + 1)), D.expand(k, -1, -1), Hr], 1)
            one = torch.ones(k, 1, dtype=F64, device=DEV)
            b = torch.cat([torch.where(on, Bf, 1.0).repeat(1, p + 1), VMAX * one.expand(k, 6 * p),
                           AMAX * one.expand(k, 6 * (p - 1)), hr], 1)
            Ac = A[:, :, free].contiguous()
            bc = b - (A @ y0[..., None])[..., 0]
            H = 2 * Q3[free, free]
            g = 2 * (y0 @ Q3)[:, free]
            if free.stop == free.start:
                continue
            bi = torch.where((Ac.norm(dim=-1) < 1e-12) & (bc > -1e-9), 1.0, bc)
            _, act, live, ok = _ipm(H, g.detach(), Ac, bi.detach())
            xs = _kkt(H, g, Ac, bc, act, live)
            ok &= torch.isfinite(xs).all(1)
            y = torch.cat([y0[:, :free.start], xs, y0[:, free.stop:]], 1)
            f = (y * (y @ Q3)).sum(1)
            w = 3 * pt[i][:, None] + torch.arange(3 * (p + 1), device=DEV)
            P[w[ok]] = y[ok].detach()
            cost[i[ok]] = f[ok].detach()
            if gP is not None and n <= 512:
                loss = ((y * gP[w]).sum(1) + f)[ok].sum()
                a, c, e = torch.autograd.grad(loss, (X, Z, Bf))
                gx[i[ok]], gg[i[ok]] = a[ok], c[ok]
                to = fo[i][:, None] + j
                e = e * ok[:, None]
                gb[to[on]] = e[on]
    res = dict(P=P, cost=cost, status=None)
    if gP is not None and n > 512:
        # the derivative jumps where a row is only just active: among thousands of
        # edges some are, and this method and the library's may take either side
        gx = gg = gb = None
        res.update(grad_x0=None, grad_goal=None, grad_b=None)
        if case["use"] == "solve_backward":
            res["flags"] = None
    elif case["use"] == "solve_backward":
        res.update(grad_x0=gx, grad_goal=gg, grad_b=gb, flags=None)
    elif case["use"] == "autograd":
        idx = torch.cat([torch.arange(int(a), int(a) + int(k)) for a, k in zip(po[pi].tolist(), nf.tolist())]).to(DEV)
        res.update(grad_x0=gx, grad_goal=gg, grad_b=torch.zeros_like(bf).index_add_(0, idx, gb))
    return res


def _exact_paths(case, seed):
    q, x0, goal = _path_inputs(case, seed)
    p, n = 7, case["n"]
    so = torch.as_tensor(q.seg_off, device=DEV)
    S = so[1:] - so[:-1]
    po = torch.as_tensor(q.poly_off, dtype=torch.int64, device=DEV)
    nf = po[1:] - po[:-1]
    fcap = int(nf.max())
    Af, bf = torch.as_tensor(q.A_face, device=DEV), torch.as_tensor(q.b_face, device=DEV)
    H = torch.as_tensor(q.H, device=DEV).reshape(-1, 32, 24)
    h0, G = torch.as_tensor(q.h0, device=DEV).reshape(-1, 32), torch.as_tensor(q.G, device=DEV).reshape(-1, 32, 6)
    P = torch.full((int(so[-1]), 24), float("nan"), dtype=F64, device=DEV)
    cost = torch.full((n,), float("inf"), dtype=F64, device=DEV)
    V, W = _derivative_rows(p)
    D = _kron3(np.concatenate([V, -V, W, -W]))
    Q = _bernstein_cost(p)
    eye3 = torch.eye(3, dtype=F64, device=DEV)
    for s in torch.unique(S).tolist():
        # control points of every segment from the 5 s + 3 that are free of the joins
        M = np.zeros((s, 8, 5 * s + 3))
        M[0, :, :8] = np.eye(8)
        for t in range(1, s):
            a, b, c = M[t - 1, 5], M[t - 1, 6], M[t - 1, 7]
            M[t, 0], M[t, 1], M[t, 2] = c, 2 * c - b, 4 * c - 4 * b + a
            for k in range(5):
                M[t, 3 + k, 8 + 5 * (t - 1) + k] = 1.0
        Mt = torch.as_tensor(M, dtype=F64, device=DEV)
        M3 = torch.stack([torch.kron(Mt[t], eye3) for t in range(s)])          # [s, 24, 3(5s+3)]
        Qg = torch.kron(sum(Mt[t].T @ Q @ Mt[t] for t in range(s)), eye3)
        nv = 3 * (5 * s + 3)
        free = slice(3, nv - 3)
        E = torch.zeros(6, 24, dtype=F64, device=DEV)                          # join state of a segment
        E[:3, :3] = eye3
        E[3:, :3], E[3:, 3:6] = -p * eye3, p * eye3
        for i in torch.split(torch.nonzero(S == s)[:, 0], max(16, 1600 // (s * s))):
            k = len(i)
            seg = so[i][:, None] + torch.arange(s, device=DEV)
            j = torch.arange(fcap, device=DEV)
            on = j < nf[seg][..., None]
            at = (po[seg][..., None] + j).clamp_max(len(bf) - 1)
            An, Bn = Af[at] * on[..., None], torch.where(on, bf[at], 1.0)
            rows, rhs = [], []
            for t in range(s):
                Fr = torch.zeros(k, 8, fcap, 8, 3, dtype=F64, device=DEV)
                for u in range(8):
                    Fr[:, u, :, u] = An[:, t]
                Hs, hs = H[seg[:, t]], h0[seg[:, t]]
                if t == 0:
                    hs = hs + (G[seg[:, t]] * x0[i][:, None]).sum(-1)
                else:
                    Hs = Hs - G[seg[:, t]] @ E
                L = torch.cat([Fr.reshape(k, -1, 24), D.expand(k, -1, -1), Hs], 1)
                rows.append(L @ M3[t])
                rhs.append(torch.cat([Bn[:, t].repeat(1, 8), torch.full((k, 42), VMAX, dtype=F64, device=DEV),
                                      torch.full((k, 36), AMAX, dtype=F64, device=DEV), hs], 1))
            A, b = torch.cat(rows, 1), torch.cat(rhs, 1)
            y0 = torch.zeros(k, nv, dtype=F64, device=DEV)
            y0[:, :3], y0[:, -3:] = x0[i, :3], goal[i]
            Ac, bc = A[:, :, free].contiguous(), b - (A @ y0[..., None])[..., 0]
            bc = torch.where((Ac.norm(dim=-1) < 1e-12) & (bc > -1e-9), 1.0, bc)
            Hq, g = 2 * Qg[free, free], 2 * (y0 @ Qg)[:, free]
            _, act, live, ok = _ipm(Hq, g, Ac, bc)
            y = y0.clone()
            y[:, free] = _kkt(Hq, g, Ac, bc, act, live, 1e-13)
            ok &= torch.isfinite(y).all(1)
            P[seg[ok]] = torch.einsum("srv,kv->ksr", M3, y)[ok]
            cost[i[ok]] = (y * (y @ Qg)).sum(1)[ok]
    return dict(P=P.reshape(-1), cost=cost, status=None)


def _exact_mpc(case, seed):
    q, x0, ref, planes = _mpc_inputs(case, seed)
    n, N, dt = case["n"], case["N"], q.dt
    I3 = np.eye(3)
    A = np.block([[I3, dt * I3], [0 * I3, I3]])
    B = np.concatenate([dt * dt / 2 * I3, dt * I3])
    Sx, Su = np.zeros((N + 1, 6, 6)), np.zeros((N + 1, 6, 3 * N))
    Sx[0] = np.eye(6)
    for k in range(N):
        Sx[k + 1] = A @ Sx[k]
        Su[k + 1] = A @ Su[k]
        Su[k + 1][:, 3 * k:3 * k + 3] += B
    Eu, Ev = np.linalg.svd(Su[N])[::2]
    Z = torch.as_tensor(Ev[6:].T, dtype=F64, device=DEV)                       # inputs that do not move x_N
    pinv = torch.as_tensor(np.linalg.pinv(Su[N]), dtype=F64, device=DEV)
    Sx, Su = torch.as_tensor(Sx, device=DEV), torch.as_tensor(Su, device=DEV)
    Qm, F1, F2, G = (torch.as_tensor(v, dtype=F64, device=DEV) for v in (q.Q, q.F1, q.F2, q.G))
    Hu = 2 * 0.01 * torch.eye(3 * N, dtype=F64, device=DEV)
    for k in range(1, N):
        Hu += 2 * Su[k].T @ Qm @ Su[k]
    d = (Su[1:] - Su[:-1])[:, :3]
    Hu += 2 * q.w * (d.transpose(1, 2) @ d).sum(0)
    fixed = torch.cat([F1 @ Su[k] + F2 @ Su[k + 1] for k in range(N)])
    X = torch.full((n, N + 1, 6), float("nan"), dtype=F64, device=DEV)
    U = torch.full((n, N, 3), float("nan"), dtype=F64, device=DEV)
    cost = torch.full((n,), float("inf"), dtype=F64, device=DEV)
    for i in torch.split(torch.arange(n, device=DEV), 64):
        k = len(i)
        xf = torch.einsum("tab,kb->kta", Sx, x0[i])                            # free motion
        up = (ref[i, N] - xf[:, N]) @ pinv.T
        xp = xf + torch.einsum("tau,ku->kta", Su, up)
        dev = (xp - ref[i])[:, 1:N]
        gu = 2 * 0.01 * up + 2 * torch.einsum("kta,tau->ku", dev @ Qm, Su[1:N])
        gu = gu + 2 * q.w * torch.einsum("kta,tau->ku", xp[:, 1:, :3] - xp[:, :-1, :3], d)
        nk, lk = planes[i, :, :3], planes[i, :, 3]
        rows, rhs = [(fixed @ Z).expand(k, -1, -1)], [
            (G - torch.einsum("ma,kta->ktm", F1, xp[:, :-1]) - torch.einsum("ma,kta->ktm", F2, xp[:, 1:])).reshape(k, -1)]
        for pos, h in ((0, 0.0), (0, dt / 3), (1, -dt / 3), (1, 0.0)):
            Mj = (Su[pos:pos + N, :3] + h * Su[pos:pos + N, 3:]) @ Z           # [N, 3, nz]
            pj = xp[:, pos:pos + N, :3] + h * xp[:, pos:pos + N, 3:]
            rows.append(-torch.einsum("ktc,tcz->ktz", nk, Mj))
            rhs.append((nk * pj).sum(-1) - lk)
        H, g = Z.T @ Hu @ Z, gu @ Z
        A_, b_ = torch.cat(rows, 1), torch.cat(rhs, 1)
        b_ = torch.where((A_.norm(dim=-1) < 1e-10) & (b_ > -1e-9), 1.0, b_)
        _, act, live, ok = _ipm(H, g, A_, b_)
        u = up + _kkt(H, g, A_, b_, act, live, 1e-13) @ Z.T
        ok &= torch.isfinite(u).all(1)
        x = xf + torch.einsum("tau,ku->kta", Su, u)
        X[i[ok]], U[i[ok]] = x[ok], u.reshape(k, N, 3)[ok]
        dev = (x - ref[i])[:, 1:N]
        f = ((dev @ Qm) * dev).sum((1, 2)) + 0.01 * (u * u).sum(1)
        f = f + q.w * ((x[:, 1:, :3] - x[:, :-1, :3]) ** 2).sum((1, 2))
        cost[i[ok]] = f[ok]
    return dict(X=X, U=U, cost=cost, status=None)


def exact(case, seed):
    kind = case["kind"]
    if kind == "segments":
        return _exact_segments(case, seed)
    if kind == "paths":
        # the dense interior point takes too long on many long paths
        return _exact_paths(case, seed) if case["n"] * case["s_hi"] ** 2 <= 160_000 else None
    if kind == "mpc":
        return _exact_mpc(case, seed) if case["n"] * case["N"] ** 2 <= 1_500_000 else None
    if kind == "planes":
        R = _Rand(seed)
        lo, hi = _boxes(R, case["boxes"])
        X = R.uniform(0.0, 10.0, case["n"], 3)
        c = torch.minimum(torch.maximum(X[:, None], lo), hi)
        i = ((X[:, None] - c) ** 2).sum(-1).argmin(1)
        pt = c[torch.arange(len(X), device=DEV), i]
        d = X - pt
        nn = d.norm(dim=1, keepdim=True)
        nrm = torch.where(nn > 0, d / nn.clamp_min(1e-300), 0.0)
        return dict(index=None, point=pt, plane=torch.cat([nrm, (nrm * pt).sum(1, keepdim=True)], 1))
    return None   # whole numbers and bytes, and the Cut-QP's values, which have no closed form
