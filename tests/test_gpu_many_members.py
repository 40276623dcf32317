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


@pytest.mark.parametrize("copies", [100, 110])
def test_members_round_alike_in_a_batch_of_hundreds(copies):
    """500 and 550 members whose first coarse levels have some 40 to 330 rows: with more
    than 512 their workgroups are smaller; bit for bit as each member alone."""
    need_gpu()
    from paper_1910_11463_amd.solver import Amg
    from tests.test_gpu_tail import _batch, _even
    opts = dict(tol_inner=1e-11, max_inner=400, coarse_max=16, relax_pre_coarse="FC", relax_post_coarse="C")
    sizes = [130, 190, 200, 760, 1000]
    mats = [_even(n, 3, n) for n in sizes]
    b = [np.random.default_rng(n).uniform(-1.0, 1.0, n) for n in sizes]
    rowptr, col, val, seg = _batch(mats * copies)
    a = Amg(**opts)
    a.setup(rowptr, col, val, seg)
    x, it, rel, rc = a.solve(np.concatenate(b * copies))
    a.close()
    assert rc == 0, rel
    for s, m in enumerate(mats):
        one = Amg(**opts)
        one.setup(*m)
        print("member of", sizes[s], "rows, coarse", len(one.level(1)["rowptr"]) - 1, flush=True)
        y, it1, _, rc1 = one.solve(b[s])
        one.close()
        assert rc1 == 0
        for k in range(s, len(sizes) * copies, len(sizes)):
            assert it[k] == it1[0] and np.array_equal(x[seg[k]:seg[k + 1]], y), k
