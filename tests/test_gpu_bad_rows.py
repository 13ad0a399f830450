"""A reachable row with one coefficient that is not finite makes its edge invalid input,
whichever coefficient it is (start, interior or goal point), also with the start at
the origin, where the row's bound takes every coefficient times 0."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", range(3, 10))
@pytest.mark.parametrize("at_origin", [False, True])
def test_every_column(p, at_origin):
    from tests.test_gpu_near_parallel import _instances, _solve
    from workloads import gen
    base = _instances(p, n=1)[0]
    H, h0, G = gen._reach_block(np.random.default_rng(p), 100, p, 0.9, 2.6)
    base.update(H=H, h0=h0, G=G)
    if at_origin:
        base["x0"] = np.zeros(6)
    insts = [base]
    for col in range(3 * (p + 1)):
        for row, v in ((0, np.nan), (63, np.inf), (64, -np.inf), (99, np.nan)):
            K = H.copy()
            K[row, col] = v
            insts.append(dict(base, H=K))
    for iters in (0, None):
        st, P, _ = _solve(insts, iters)
        assert st[0] != 5 and (st[1:] == 5).all(), np.flatnonzero(st[1:] != 5)
        assert np.isnan(P[1:]).all()
