"""Gradients of solved instances alone, face offsets among them, from working sets
reached through different warm starts: the derivative uses the factor that the
forward pass kept (basis and packed R^-1)."""
import numpy as np
import pytest

from tests.test_gpu_working_set import _instances

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,r", [(3, 64), (3, 128), (5, 1), (5, 65), (7, 32), (8, 0), (8, 128), (9, 32), (9, 65)])
def test_same_gradients_from_any_warm_start(p, r):
    import torch
    from paper_2411_13507_amd import _lib
    from paper_2411_13507_amd.api import SegmentBatchGPU
    b = _instances(p, r, 96)
    gb = SegmentBatchGPU(b)
    x0, goal = torch.as_tensor(b.x0, device="cuda"), torch.as_tensor(b.goal, device="cuda")
    gP = torch.as_tensor(np.random.default_rng(p).standard_normal(3 * gb.points_total), device="cuda")
    gf = torch.ones(b.n, dtype=torch.float64, device="cuda")

    def solve(iters, rho):
        o = _lib.default_opts()
        o.admm_iters, o.rho = iters, rho
        res = gb.solve(x0, goal, opts=o)
        g = gb.backward(gP, gf)
        f = g.b_inst.cpu().numpy()
        rows = [np.concatenate([g.x0[i].cpu().numpy(), g.goal[i].cpu().numpy(), f[gb.face_off[i]:gb.face_off[i + 1]]])
                for i in range(b.n)]
        return res.status.cpu().numpy() == 0, g.flags.cpu().numpy() == 0, rows

    ok, clean, ref = solve(0, 0.1)
    for iters, rho in ((3, 30.0), (10, 0.1), (40, 0.1)):
        ok2, clean2, got = solve(iters, rho)
        assert np.array_equal(ok2, ok)
        use = np.flatnonzero(ok & clean & clean2)
        assert len(use) >= 5 or r > 64
        # 1e-6 relative, as derivatives of optima that agree to 1e-8 or better; a row that
        # is only just active may be in one working set and not in the other
        same = [np.linalg.norm(got[i] - ref[i]) <= 1e-6 * (1 + np.linalg.norm(ref[i])) for i in use]
        print(f"case: p {p}, r {r}, {iters} iterations: {sum(same)} of {len(use)} solved instances agree", flush=True)
        assert len(use) and np.mean(same) >= 0.9
