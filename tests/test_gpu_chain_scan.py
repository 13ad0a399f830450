"""Path solve at the edges of its scan, its products with L^-1 and its launches
(one wavefront per path with a small working-set cap, four with the full one):
one, two, three and twelve segments, polytopes with more than 32 faces, no, more
than 32 and more than 64 reachable rows per segment, another duration, and the
largest LDS footprint, against the FP64 oracle at the tolerances of the other path
tests.  Each batch is solved as it is and tiled to more paths than are taken
with four wavefronts from the start: copies must agree bit for bit."""
import dataclasses

import numpy as np
import pytest
from scipy.optimize import linprog

from tests.test_gpu_chains import _opts, compare_chains, gpu_chains
from workloads import gen

pytestmark = pytest.mark.gpu


def _middle(A, b):
    """Centre of the largest ball in {x: A x <= b}."""
    r = linprog([0, 0, 0, -1], np.c_[A, np.linalg.norm(A, axis=1)], b, bounds=[(None, None)] * 3 + [(0, None)])
    return r.x[:3]


def _pick(b, paths, S=None, faces=None, T=None, bare=False):
    """The first S segments of some paths of ``b`` (the goal then the middle of the
    last one's polytope), every polytope padded to ``faces`` faces with looser copies
    of its own; ``bare`` leaves reachable rows to the first path alone (the call wants
    some)."""
    seg_off, A, f, po, H, h0, G, ro, ho, x0, goal = [0], [], [], [0], [], [], [], [0], [0], [], []
    for c in paths:
        ch = b.chain(c)
        segs = ch["segments"] if S is None else ch["segments"][:S]
        for s in segs:
            a, bb = s["A_face"], s["b_face"]
            if faces is not None:
                k = np.arange(faces - len(bb)) % len(bb)
                a, bb = np.concatenate([a, a[k]]), np.concatenate([bb, bb[k] + 0.1])
            A.append(a); f.append(bb); po.append(po[-1] + len(bb))
            r = 0 if bare and c != paths[0] else len(s["h0"])
            H.append(s["H"][:r].ravel()); h0.append(s["h0"][:r]); G.append(s["G"][:r])
            ro.append(ro[-1] + r); ho.append(ho[-1] + H[-1].size)
        seg_off.append(seg_off[-1] + len(segs))
        goal.append(ch["goal"] if S is None else _middle(segs[-1]["A_face"], segs[-1]["b_face"]))
        x0.append(ch["x0"])
    return dataclasses.replace(
        b, T=b.T if T is None else T, seg_off=np.asarray(seg_off, np.int64), poly_off=np.asarray(po, np.int32),
        A_face=np.concatenate(A), b_face=np.concatenate(f), poly_idx=np.arange(len(A), dtype=np.int32),
        reach_off=np.asarray(ro, np.int64), H_off=np.asarray(ho, np.int64), H=np.concatenate(H),
        h0=np.concatenate(h0), G=np.concatenate(G).reshape(-1, 6), x0=np.asarray(x0), goal=np.asarray(goal))


def _longest(b, n):
    return [int(c) for c in np.argsort(-np.diff(b.seg_off), kind="stable")[:n]]


CASES = {
    "one": dict(S=1), "two": dict(S=2), "three": dict(S=3), "longest": dict(),
    "faces33": dict(faces=33, S=4), "faces64": dict(faces=64, S=5),
    "reach0": dict(bare=True, S=4), "reach33": dict(r=33, S=5), "reach70": dict(r=70, S=4),
    "T1.3": dict(T=1.3, S=6), "lds": dict(r=128, faces=64),
}


@pytest.mark.parametrize("admm", [0, None], ids=["polish-only", "default"])
@pytest.mark.parametrize("name", CASES)
def test_chain_edges(gpu_available, name, admm):
    kw = dict(CASES[name])
    n = 4 if name == "lds" else 8
    src = gen.gen_cfg3(indices=range(48), r=kw.pop("r", 32))
    b = _pick(src, _longest(src, n), **kw)
    print(f"case: {name}, {b.n} paths, admm_iters {admm}", flush=True)
    _, out = gpu_chains(b, _opts(admm))
    compare_chains(b, out, list(range(b.n)), name)
    copies = 1152 // b.n                           # more than four paths per CU
    _, big = gpu_chains(gen.concat_chains([b] * copies), _opts(admm))
    for k in ("status", "cost"):
        t = big[k].reshape(copies, -1)
        assert np.array_equal(t, np.broadcast_to(t[0], t.shape), equal_nan=(k == "cost")), k
    t = big["P"].reshape(copies, -1)
    assert np.array_equal(t, np.broadcast_to(t[0], t.shape), equal_nan=True)
    compare_chains(b, dict(P=t[0], status=big["status"][:b.n], cost=big["cost"][:b.n], kkt=big["kkt"][:b.n]),
                   list(range(b.n)), name + " tiled")
