"""Short horizons in batches of more than three per compute unit are solved by one
wavefront each instead of four: the same results, bit for bit, as in a small batch,
at the edges of the rule (passes of 64 rows, plane rows past the last of them)."""
import numpy as np
import pytest

from tests.test_gpu_mpc import run
from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,extra", [(2, 0), (2, 20), (3, 9), (3, 10), (4, 20), (5, 0), (6, 20), (7, 15), (7, 16),
                                     (8, 4), (12, 4), (16, 0), (17, 0)])
def test_as_in_a_small_batch(N, extra):
    import torch
    b = gen.gen_mpc(n=40, N=N, m_extra=extra)
    b.planes[5, N // 2, 3] += 5.0 * np.linalg.norm(b.planes[5, N // 2, :3])   # one that cannot hold
    small = run(b)
    n = 3 * torch.cuda.get_device_properties(0).multi_processor_count + 7
    at = np.arange(n) % b.n
    large = run(b.subset(at))
    print(f"case: N {N}, {12 + extra} rows, statuses {np.unique(small['status'], return_counts=True)}", flush=True)
    for k, v in large.items():
        assert np.array_equal(v, small[k][at], equal_nan=True), k
