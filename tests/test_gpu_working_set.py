"""The working set's factor is kept as an orthonormal basis and R^-1, appended
to and rotated as rows enter and leave.  Warm starts that propose poor working
sets (few iterations, extreme penalties) make the polish drop many rows; the
optimum must not depend on them.  Degrees 3 and 9 are the smallest and largest
factors (6 and 24 rows), 0, 64 and 128 reachable rows the edges of the lanes'
row slots."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _instances(p, r, n=24):
    from workloads import gen
    out = []
    for i in range(n):
        rng = np.random.default_rng([p, r, i])
        c = rng.uniform(2, 8, 3)
        nf = int(rng.integers(6, 41))
        A, b, w = gen._box_polytope(rng, nf, c)
        s = gen._sample_in(rng, A, b, c, w)
        g = gen._sample_in(rng, A, b, c, w)
        # (a batch holds at least one reachable row: H may not be empty)
        H, h0, G = gen._reach_block(rng, r if i else max(r, 1), p, 1.3, 3.3)
        out.append(dict(p=p, T=1.0, vmax=3.0, amax=5.0, A_face=A, b_face=b, H=H, h0=h0, G=G,
                        x0=np.concatenate([s, rng.uniform(-1, 1, 3)]), goal=g))
    return gen.from_instances(out)


@pytest.mark.parametrize("p", [3, 5, 7, 8, 9])
@pytest.mark.parametrize("r", [0, 1, 32, 64, 65, 128])
def test_same_optimum_from_any_warm_start(p, r):
    import torch
    from paper_2411_13507_amd import _lib
    from paper_2411_13507_amd.api import SegmentBatchGPU
    b = _instances(p, r)
    gb = SegmentBatchGPU(b)
    x0, goal = torch.as_tensor(b.x0, device="cuda"), torch.as_tensor(b.goal, device="cuda")
    gP = torch.as_tensor(np.random.default_rng(p).standard_normal(3 * gb.points_total), device="cuda")
    gf = torch.ones(b.n, dtype=torch.float64, device="cuda")

    def solve(iters, rho):
        o = _lib.default_opts()
        o.admm_iters, o.rho = iters, rho
        res = gb.solve(x0, goal, opts=o)
        g = gb.backward(gP, gf)
        return [t.cpu().numpy() for t in (res.status, res.cost, res.P, g.x0, g.goal, g.b_inst, g.flags)]

    ref = solve(0, 0.1)
    ok = ref[0] == 0
    assert set(np.unique(ref[0])) <= {0, 1} and (ok.any() or r > 32)
    for iters, rho in ((1, 0.1), (3, 30.0), (10, 1e-3), (40, 0.1)):
        got = solve(iters, rho)
        assert np.array_equal(got[0], ref[0])
        # both are the optimum to the polish's tolerance (1e-11 relative on rows)
        assert np.allclose(got[1][ok], ref[1][ok], rtol=1e-8, atol=1e-9)
        assert np.allclose(got[2], ref[2], rtol=0, atol=1e-8, equal_nan=True)
        clean = (got[6] == 0) & (ref[6] == 0)
        for a, c in ((got[3], ref[3]), (got[4], ref[4])):
            d = np.linalg.norm(a - c, axis=1)[clean]
            # a row that is only just active may be in one working set and not
            # in the other: nearly all gradients agree, to 1e-6 relative
            assert (d <= 1e-6 * (1 + np.linalg.norm(c, axis=1)[clean])).mean() >= 0.9
