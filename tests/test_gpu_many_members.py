"""The generic solver on tens of thousands of small segments."""
import time

import numpy as np
import pytest

from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu


def _chains(k, n):
    """k unsymmetric tridiagonal matrices of n rows, diagonally dominant."""
    j = np.arange(k * n) % n
    i = np.arange(k * n)
    has = np.stack([j > 0, np.ones(k * n, bool), j < n - 1], 1)
    rng = np.random.default_rng(k)
    cols = np.stack([i - 1, i, i + 1], 1)
    vals = np.stack([-0.6 * rng.uniform(0.5, 1.0, k * n), np.ones(k * n), -0.2 * rng.uniform(0.5, 1.0, k * n)], 1)
    rowptr = np.concatenate([[0], np.cumsum(has.sum(1))]).astype(np.int64)
    return rowptr, cols[has].astype(np.int32), vals[has], np.arange(k + 1, dtype=np.int64) * n


def test_setup_time_grows_with_the_number_of_segments():
    """Four times the segments: about 3.5 times the time (12.7 times where each
    segment walked the list of all before it)."""
    need_gpu()
    from paper_1910_11463_amd.solver import Amg
    best = []
    for k in (8000, 32000):
        m = _chains(k, 40)
        a = Amg(coarse_max=16)
        t = []
        for _ in range(4):
            t0 = time.perf_counter()
            a.setup(*m)
            t.append(time.perf_counter() - t0)
        a.close()
        best.append(min(t))
    print("seconds", best, flush=True)
    assert best[1] < 7.0 * best[0]
