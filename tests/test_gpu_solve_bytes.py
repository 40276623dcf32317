"""stats.bytes_solve against the bytes of the kernels that run, counted from the
hierarchy's matrices: levels of the level kernels (whose first half-sweep is part of
the restriction) and levels in the tail (packed entries of 10 bytes)."""
import numpy as np
import pytest

from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu


def _half(nF, nC, zF, zC, ch):
    return (nF, zF) if ch == "F" else (nC, zC)


@pytest.mark.parametrize("n", [5, 14])
@pytest.mark.parametrize("pre,post", [("FC", "FC"), ("C", "FF"), ("", "F")])
def test_bytes_per_cycle(n, pre, post):
    need_gpu()
    from paper_1910_11463_amd import workloads as wl
    from paper_1910_11463_amd.solver import Amg, Solver
    om, w = Solver.level_symmetric(4)
    mesh = wl.hex_mesh(n)
    opts = dict(relax_pre="FC", relax_post="F", relax_pre_coarse=pre, relax_post_coarse=post, max_inner=200)
    s = Solver(**opts)
    s.set_mesh(mesh)
    s.set_quadrature(om[5:6], np.array([4.0 * np.pi]))
    rng = np.random.default_rng(n)
    st = np.exp(rng.uniform(np.log(0.1), np.log(10.0), s.E))
    s.set_materials(st, 0.5 * st, np.ones(s.E))
    stats = s.transport_sweep(want_psi=False)[2]
    rp, col, val, _ = s.export_fine_operator(0, with_rhs=False)
    s.close()
    a = Amg(**opts)
    a.setup(rp, col, val)
    lev = [a.level(l) for l in range(a.num_levels())]
    a.close()
    N, E = len(rp) - 1, mesh.n_elem
    sizes = [len(L["rowptr"]) - 1 for L in lev]
    assert sizes == stats["level_n"][:len(lev)]
    # the levels that one workgroup takes: at most 2048 rows and 65536 padded entries
    # there and further down (here no level is near that limit)
    entries = [len(L["col"]) for L in lev]
    assert all(z < 40000 or z > 65536 for z in entries)
    tail = [l >= 1 and max(sizes[l:]) <= 2048 and max(entries[l:]) < 40000 for l in range(len(lev))]
    assert any(tail[:-1])
    total = 0.0
    for l, L in enumerate(lev[:-1]):
        m, nc, z, zr = sizes[l], sizes[l + 1], len(L["col"]), len(L["r_col"])
        lens = np.diff(L["rowptr"])
        F = L["cf"] < 0
        part = lambda ch: _half(F.sum(), m - F.sum(), lens[F].sum(), lens[~F].sum(), ch)
        if tail[l]:
            read = z + zr + sum(part(ch)[1] for ch in (pre[1:] + post))
            total += 10.0 * read + 12.0 * m + 2.0 * nc + (0.0 if tail[l - 1] else 16.0 * m)
            continue
        if l == 0:       # factored elements
            total += sum(8.0 * part(ch)[0] + 16.0 * m + 8.0 * E + m / 8.0 for ch in "FCF")
            total += 24.0 * m + 8.0 * E
        else:
            total += 8.0 * m if not pre else 8.0 * part(pre[0])[0] + 9.0 * m
            for ch in pre[1:] + post:
                k, e = part(ch)
                total += 12.0 * e + 24.0 * k + 19.0 * m
            total += 12.0 * z + 34.0 * m
        total += 12.0 * zr + 16.0 * nc + 8.0 * m + 2.0 * nc      # restriction
        total += 22.0 * m + 8.0 * nc                             # interpolation
    total += 8.0 * sizes[-1] ** 2 + 16.0 * sizes[-1]
    total += 16.0 * N + 8.0 * E                                  # convergence test
    got = stats["bytes_solve"] / stats["vcycles_total"]
    print("bytes per cycle", got, total, sizes, flush=True)
    assert abs(got - total) <= 1e-12 * total
