"""The small levels of a V-cycle in one launch (at most 2048 rows of a member on
the first of them): sizes around that limit, members of different depth in one
batch, every schedule, and rows of many lengths."""
import numpy as np
import pytest

from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu


def _matrix(n, fill, seed):
    """A diagonally dominant random matrix (CSR) with rows of very different
    lengths; 1 / (1 - 0.8) bounds its inverse in the maximum norm."""
    rng = np.random.default_rng(seed)
    rows, cols, vals = [], [], []
    for i in range(n):
        k = int(min(n - 1, rng.integers(0, fill) * rng.integers(0, 3)))
        c = np.unique(rng.integers(0, n, size=k))
        c = c[c != i]
        v = rng.uniform(0.1, 1.0, len(c))
        if len(c):
            v *= -0.8 / v.sum()
        c = np.append(c, i)
        v = np.append(v, 1.0)
        o = np.argsort(c)
        rows.append(np.full(len(c), i))
        cols.append(c[o])
        vals.append(v[o])
    rowptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    return rowptr, np.concatenate(cols).astype(np.int32), np.concatenate(vals)


def _batch(mats):
    rp, ci, va, seg = [np.zeros(1, np.int64)], [], [], [0]
    for rowptr, col, val in mats:
        rp.append(rowptr[1:] + rp[-1][-1])
        ci.append(col + seg[-1])
        va.append(val)
        seg.append(seg[-1] + len(rowptr) - 1)
    return np.concatenate(rp), np.concatenate(ci).astype(np.int32), np.concatenate(va), seg


def _dense(m):
    rowptr, col, val = m
    n = len(rowptr) - 1
    A = np.zeros((n, n))
    A[np.repeat(np.arange(n), np.diff(rowptr)), col] = val
    return A


# finest levels from one row up to past the limit: the tail starts on the first
# coarse level of the small ones, further down or nowhere for the others
SIZES = [1, 63, 64, 65, 130, 700, 2047, 2300]


@pytest.mark.parametrize("pre,post", [("FC", "FC"), ("F", ""), ("FFC", "C"), ("", "F")])
@pytest.mark.parametrize("fp32", [0, 1])
def test_members_of_every_size(pre, post, fp32):
    """Every member alone and in one batch: the same iterates bit for bit, and the
    dense solution (tol_inner 1e-11 times 5, the bound of the inverse, times the
    ratio of the norms, below sqrt(2300) = 48)."""
    need_gpu()
    from paper_1910_11463_amd.solver import Amg
    mats = [_matrix(n, 14, n) for n in SIZES]
    opts = dict(tol_inner=1e-11, max_inner=400, relax_pre="FC", relax_post="FC", relax_pre_coarse=pre,
                relax_post_coarse=post, coarse_fp32=fp32)
    rng = np.random.default_rng(5)
    b = [rng.uniform(-1.0, 1.0, n) for n in SIZES]
    rowptr, col, val, seg = _batch(mats)
    a = Amg(**opts)
    a.setup(rowptr, col, val, seg)
    x, it, rel, rc = a.solve(np.concatenate(b))
    assert rc == 0, rel
    for s, m in enumerate(mats):
        one = Amg(**opts)
        one.setup(*m)
        y, it1, _, rc1 = one.solve(b[s])
        assert rc1 == 0 and it1[0] == it[s]
        assert np.array_equal(x[seg[s]:seg[s + 1]], y), SIZES[s]
        ref = np.linalg.solve(_dense(m), b[s])
        assert np.abs(y - ref).max() <= 1e-11 * 5 * 48 * max(1.0, np.abs(b[s]).max()) + 1e-13
        one.close()
    a.close()


def _even(n, m, seed):
    """As _matrix, every row with m random columns."""
    rng = np.random.default_rng(seed)
    A = np.zeros((n, n))
    A[np.arange(n)[:, None], rng.integers(0, n, (n, m))] = -rng.uniform(0.1, 1.0, (n, m))
    np.fill_diagonal(A, 0.0)
    A *= 0.8 / np.abs(A).sum(1, keepdims=True)
    np.fill_diagonal(A, 1.0)
    rows, cols = np.nonzero(A)
    return np.concatenate([[0], np.cumsum(np.bincount(rows))]).astype(np.int64), cols.astype(np.int32), A[rows, cols]


@pytest.mark.parametrize("n,m,long_rows", [(2000, 3, False), (3000, 20, True)])
def test_levels_of_long_rows_stay_with_the_level_kernels(n, m, long_rows):
    """A member whose first coarse level has some 400 rows of over 200 entries: its
    half-sweeps there are launches of their own (one workgroup takes longer), those of a
    member of short rows are not; alone, beside another and against the dense solution
    (bound as above, with sqrt(3000) = 55)."""
    import ctypes
    need_gpu()
    from paper_1910_11463_amd import binding as B
    from paper_1910_11463_amd.solver import Amg
    mat = _even(n, m, n)
    opts = dict(tol_inner=1e-11, max_inner=400, use_graph=0)
    b = np.random.default_rng(9).uniform(-1.0, 1.0, n)
    one = Amg(**opts)
    one.setup(*mat)
    L1 = one.level(1)
    print("first coarse level", len(L1["rowptr"]) - 1, len(L1["col"]), flush=True)
    assert len(L1["rowptr"]) - 1 <= 2048 and (len(L1["col"]) > 60000) == long_rows
    B.check(B.pair_profile_enable(1))
    y, it, rel, rc = one.solve(b)
    k, ms, by = ctypes.c_int64(), ctypes.c_double(), ctypes.c_double()
    B.check(B.pair_profile_read(3, ctypes.byref(k), ctypes.byref(ms), ctypes.byref(by)))
    B.check(B.pair_profile_enable(0))
    one.close()
    assert rc == 0, rel
    assert (k.value > 0) == long_rows
    assert np.abs(y - np.linalg.solve(_dense(mat), b)).max() <= 1e-11 * 5 * 55 * max(1.0, np.abs(b).max()) + 1e-13
    rowptr, col, val, seg = _batch([_even(700, 4, 7), mat])
    a = Amg(**opts)
    a.setup(rowptr, col, val, seg)
    x, it2, _, rc2 = a.solve(np.concatenate([np.ones(700), b]))
    a.close()
    assert rc2 == 0 and it2[1] == it[0] and np.array_equal(x[700:], y)
