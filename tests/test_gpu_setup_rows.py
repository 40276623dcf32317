"""The setup's row kernels (strength, strong entries, C/F split, interpolation) at
the row lengths and list sizes where their forms change, against the reference
AIR: decisions exact, so no tolerance."""
import numpy as np
import pytest
import scipy.sparse as sp

from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu


def _check(A, seed=3, coarse_max=8):
    from oracle import air_ref as AR
    from paper_1910_11463_amd.solver import Amg
    one = AR.setup(A, AR.Options(coarse_max=coarse_max, seed=seed, max_levels=2))
    assert len(one) == 2
    g = Amg(coarse_max=coarse_max, pmis_seed=seed, max_levels=2)
    g.setup(A.indptr, A.indices, A.data, None)
    got = g.level(0)
    g.close()
    assert np.array_equal(got["cf"], one[0].cf.astype(np.int8))
    assert np.array_equal(got["p"], one[0].p.astype(np.int32))
    assert np.array_equal(got["r_rowptr"], one[0].R.indptr)
    assert np.array_equal(got["r_col"], one[0].R.indices)
    return one[0]


def _of_lengths(lens, seed):
    """Rows of the given lengths: random columns, distinct magnitudes in (0.1, 1),
    a dominant diagonal."""
    rng = np.random.default_rng(seed)
    n = len(lens)
    rows, cols = [], []
    for i, m in enumerate(lens):
        c = rng.choice(n - 1, size=m - 1, replace=False)
        c = np.append(c + (c >= i), i)
        rows.append(np.full(m, i))
        cols.append(c)
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    v = -rng.uniform(0.1, 1.0, len(rows))
    v[rows == cols] = 2.0 * max(lens)
    A = sp.csr_matrix((v, (rows, cols)), shape=(n, n))
    A.sort_indices()
    return A


@pytest.mark.parametrize("lens", [(1, 2, 3, 4, 5), (15, 16), (15, 16, 17), (31, 32), (31, 32, 33), (1, 16, 33, 70)])
def test_row_lengths(lens):
    """All rows within one form, and rows of several forms in one wave; 2049 rows,
    one more than a list block takes."""
    need_gpu()
    print("row lengths", lens, flush=True)
    _check(_of_lengths([lens[i % len(lens)] for i in range(2049)], len(lens)))


@pytest.mark.parametrize("extra", [(0, 0), (0, 1), (3, 0), (5, 5)])
def test_hubs_beyond_the_packed_count(extra):
    """Strongly coupled hubs on which 2046 + extra rows depend besides each other:
    at 2047 and more the split compares the counts in full."""
    need_gpu()
    m = [2046 + e for e in extra]
    n = 2 + sum(m)
    rows = np.arange(n)
    hub = np.concatenate([[1, 0], np.repeat([0, 1], m)])
    A = sp.csr_matrix((np.concatenate([np.full(n, 4.0), np.full(n, -1.0)]),
                       (np.concatenate([rows, rows]), np.concatenate([rows, hub]))), shape=(n, n))
    A.sort_indices()
    for seed in (3, 4, 5):
        print("hubs", extra, seed, flush=True)
        L = _check(A, seed)
        assert L.cf[0] != L.cf[1]
        if m[0] != m[1]:
            assert (L.cf[0] > 0) == (m[0] > m[1])


@pytest.mark.parametrize("n", [2, 511, 2048, 2049, 5000])
def test_split_rounds_in_one_launch_and_in_lists(n):
    """A random graph of n rows around the size at which one launch runs every
    round, and above it, where only the last rounds do."""
    need_gpu()
    print("rows", n, flush=True)
    _check(_of_lengths([min(n, 2 + i % 7) for i in range(n)], n), coarse_max=min(8, n // 2))


@pytest.mark.parametrize("n,longest", [(17, 9), (2047, 16), (2049, 16), (4500, 16), (4500, 17)])
def test_coarse_operator_of_packed_rows(n, longest):
    """Rows of A P one after the other (no row of more than 16 entries; with one of 17
    they stay at their rows' places): the Galerkin operator's pattern exact, its values
    within 1e-12 of the largest, the bound of the hierarchy parity tests.  Every third
    row couples to nothing and is referred to by few rows, so that rows of A P that
    nothing needs lie between."""
    need_gpu()
    from oracle import air_ref as AR
    from paper_1910_11463_amd.solver import Amg
    print("packed rows", n, longest, flush=True)
    lens = [1 if i % 3 == 0 else min(n, 2 + i % 15) for i in range(n)]
    lens[n // 2] = min(n, longest)
    A = _of_lengths(lens, n)
    one = AR.setup(A, AR.Options(coarse_max=4, seed=3, max_levels=2))
    assert len(one) == 2 and np.diff(A.indptr).max() == max(16, longest)
    g = Amg(coarse_max=4, pmis_seed=3, max_levels=2)
    g.setup(A.indptr, A.indices, A.data, None)
    got = g.level(1)
    g.close()
    ref = one[1].A
    assert np.array_equal(got["rowptr"], ref.indptr) and np.array_equal(got["col"], ref.indices)
    assert np.abs(got["val"] - ref.data).max() <= 1e-12 * np.abs(ref.data).max()


@pytest.mark.parametrize("n,row", [(2048, 5), (2048, 60), (500, 90), (700, 50), (700, 55), (700, 60)])
def test_split_rounds_of_short_lists_with_long_rows(n, row):
    """Lists short enough for one launch, with few and with many strong entries (the
    limit of 32768 lies between 55 and 60 entries for 700 rows, five in six of them
    strong): list rounds first, then one launch."""
    need_gpu()
    print("rows", n, "of", row, flush=True)
    _check(_of_lengths([row] * n, n + row))
