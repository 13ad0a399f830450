"""The MPC solver spreads one horizon over four wavefronts: rows in passes of
64 over three of them, plane rows in the fourth, barrier Hessians six stages at
a time.  Horizons and row counts at the edges of that split (2 is the shortest
horizon; 2 m = 64, 3 passes, 5 and 6 stages, the 5- and 11-slot kernels, the
longest horizon with the most rows), against the oracle where it is quick and
by properties elsewhere."""
import numpy as np
import pytest

from tests.test_gpu_mpc import check_properties, compare, run
from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [3, 5, 6, 7, 8, 13, 20, 64])
@pytest.mark.parametrize("extra", [0, 1, 4, 9, 10, 20])
def test_split(N, extra):
    b = gen.gen_mpc(n=5, N=N, m_extra=extra)
    out = run(b)
    if N <= 8:
        from oracle import mpc as ompc
        from oracle import qp
        feas = [i for i in range(b.n) if ompc.solve(b.instance(i)).status == qp.SOLVED]
        if feas:
            compare(b, out, feas, f"N {N} m {12 + extra}")
    ok = np.flatnonzero(out["status"] == 0)
    assert len(ok) or N <= 8
    s = b.subset(ok)
    if len(ok):   # (with 20 limits on three steps nothing need be feasible)
        check_properties(s, {k: v[ok] for k, v in out.items()})
    # an instance's result does not depend on what else is in the batch
    one = run(b.subset([4]))
    for k, v in one.items():
        assert np.array_equal(v[0], out[k][4], equal_nan=True), k
