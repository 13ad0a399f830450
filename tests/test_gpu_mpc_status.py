"""Statuses of MPC horizons against the oracle, both ways, at the edges of the
split over four wavefronts (row passes, stage batches, both register-slot kernels):
what the oracle solves is solved, what the library certifies infeasible the oracle
certifies too, and what the oracle certifies infeasible is never solved."""
import multiprocessing as mp

import numpy as np
import pytest

from oracle import qp
from tests.test_gpu_mpc import _oracle, compare, run
from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [3, 5, 6, 7, 8, 13, 20, 64])
@pytest.mark.parametrize("extra", [0, 4, 9, 10, 20])
def test_both_ways(N, extra):
    b = gen.gen_mpc(n=6, N=N, m_extra=extra)
    # one horizon that cannot hold: a plane out of reach
    b.planes[5, N // 2, 3] += 5.0 * np.linalg.norm(b.planes[5, N // 2, :3])
    out = run(b)
    with mp.get_context("fork").Pool(4) as pool:
        st = np.array([o[0] for o in pool.map(_oracle, [b.instance(i) for i in range(b.n)])])
    print(f"case: N {N}, {12 + extra} rows, oracle {st.tolist()}, here {out['status'].tolist()}", flush=True)
    solved, infeasible = np.flatnonzero(st == qp.SOLVED), np.flatnonzero(st == qp.INFEASIBLE)
    assert 5 in infeasible
    if len(solved):
        compare(b, out, solved.tolist(), "solved")
    assert (st[out["status"] == qp.INFEASIBLE] == qp.INFEASIBLE).all()
    assert (out["status"][infeasible] != qp.SOLVED).all()
    assert N < 13 or len(solved) >= 4
