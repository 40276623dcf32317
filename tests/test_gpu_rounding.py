"""Rounding of the factored hex operator against a forward substitution in extended
precision (64-bit mantissa): nothing in it may add up over the elements of a sweep."""
import numpy as np
import pytest

from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu

LD, CLD = np.longdouble, np.clongdouble


def _solve(sig, kap, g):
    """[sig I + sum_d kap_d T_d]^{-1} g for elements (..., 2, 2, 2) (node axes z, y, x
    counted from the inflow side), T = M1^{-1} (upwind transport on the unit interval)
    = [[3, 1], [-3, 1]], diagonalised: eigenvalues 2 +- i sqrt 2."""
    r = np.sqrt(LD(2))
    lam = np.array([2 + 1j * r, 2 - 1j * r], dtype=CLD)
    W = np.array([[1, 1], [lam[0] - 3, lam[1] - 3]], dtype=CLD)
    det = W[0, 0] * W[1, 1] - W[0, 1] * W[1, 0]
    Wi = np.array([[W[1, 1], -W[0, 1]], [-W[1, 0], W[0, 0]]], dtype=CLD) / det

    def along(M, v, axis):
        a = np.take(v, 0, axis=axis)
        b = np.take(v, 1, axis=axis)
        return np.stack([M[0, 0] * a + M[0, 1] * b, M[1, 0] * a + M[1, 1] * b], axis=axis)

    z = g.astype(CLD)
    for ax in (-1, -2, -3):
        z = along(Wi, z, ax)
    den = (sig[..., None, None, None] + kap[2] * lam[:, None, None] + kap[1] * lam[None, :, None] +
           kap[0] * lam[None, None, :])
    z = z / den
    for ax in (-1, -2, -3):
        z = along(W, z, ax)
    return z.real


def _sweep(n, om, sig, src):
    """psi of one direction; arrays [z, y, x] and [z, y, x, 2, 2, 2]."""
    flip = [om[d] < 0 for d in range(3)]
    axes = tuple(2 - d for d in range(3) if flip[d])
    turn = lambda a: np.flip(a, axes + tuple(3 + ax for ax in axes)) if a.ndim == 6 else np.flip(a, axes)
    sig, src = turn(sig), turn(src)
    kap = [abs(LD(om[d])) * n for d in range(3)]
    x = np.zeros((n, n, n, 2, 2, 2), dtype=LD)
    k, j, i = np.meshgrid(*[np.arange(n)] * 3, indexing="ij")
    up = np.array([4, -2], dtype=LD)       # M1^{-1} times the inflow face value
    for s in range(3 * n - 2):
        K, J, I = [a[k + j + i == s] for a in (k, j, i)]
        g = src[K, J, I].copy()
        m = I > 0
        g[m] += kap[0] * x[K[m], J[m], I[m] - 1][..., 1][..., None] * up
        m = J > 0
        g[m] += kap[1] * x[K[m], J[m] - 1, I[m]][..., :, 1, :][..., None, :] * up[:, None]
        m = K > 0
        g[m] += kap[2] * x[K[m] - 1, J[m], I[m]][..., 1, :, :][..., None, :, :] * up[:, None, None]
        x[K, J, I] = _solve(sig[K, J, I], kap, g)
    return turn(x)


def test_extended_sweep_against_the_assembled_operator():
    """The reference above against the assembled operator."""
    from paper_1910_11463_amd import workloads as wl
    need_gpu()
    from tests.gpu_util import solver_for
    w = wl.make_config(2, scale=3)
    s = solver_for(w, 2)
    om, _ = s.level_symmetric(2)
    for m in (0, 5):
        rp, col, val, b = s.export_fine_operator(m)
        x = _sweep(3, om[m], w.mats.sigma_t.reshape(3, 3, 3).astype(LD),
                   np.broadcast_to((w.mats.q / (4 * np.pi)).reshape(3, 3, 3, 1, 1, 1), (3, 3, 3, 2, 2, 2)).astype(LD))
        x = x.reshape(-1).astype(np.float64)
        r = np.array([val[rp[i]:rp[i + 1]] @ x[col[rp[i]:rp[i + 1]]] for i in range(len(x))]) - b
        assert np.abs(r).max() <= 1e-13 * np.abs(b).max()
    s.close()


@pytest.mark.parametrize("n", [16, 32])
def test_sweep_error_does_not_build_up(n):
    """|psi - exact| <= 2.5e-15 |psi|, twice what the same formulas give in IEEE double on
    a CPU with sqrt 2 and its reciprocal rounded consistently (1.2e-15; with the nearest
    doubles 2.6e-15 to 3.1e-15 at n = 16 and growing with n).  Cross sections vary from
    element to element: equal ones would round alike everywhere and add up by themselves."""
    torch = need_gpu()
    from paper_1910_11463_amd import binding as B
    from paper_1910_11463_amd import workloads as wl
    from paper_1910_11463_amd.solver import Solver
    s = Solver(relax_pre="TTT", relax_post="TTT", relax_pre_coarse="F", relax_post_coarse="", tile_xy=16, filter_r=1.0,
               tol_inner=1e-10)
    s.set_mesh(wl.hex_mesh(n))
    om, w = Solver.level_symmetric(2)
    s.set_quadrature(om, w)
    rng = np.random.default_rng(n)
    st = np.exp(rng.uniform(np.log(0.1), np.log(10.0), s.E))
    ss, q, phi = 0.9 * st, rng.uniform(0.5, 1.5, s.E), rng.uniform(0.0, 1.0, s.N)
    s.set_materials(st, ss, q)
    psi, _, _, rc = s.transport_sweep(mode=B.PAIR_BATCHED, phi_in=phi)
    s.close()
    assert rc == B.PAIR_OK
    src = (ss[:, None].astype(LD) * phi.reshape(-1, 8) + q[:, None]) / (4 * np.arctan(LD(1)) * 4)
    e2 = n2 = 0.0
    for m in range(len(w)):
        ref = _sweep(n, om[m], st.reshape(n, n, n).astype(LD), src.reshape(n, n, n, 2, 2, 2)).reshape(-1)
        d = psi[m] - ref
        e2 += float((d * d).sum())
        n2 += float((ref * ref).sum())
    err = (e2 / n2) ** 0.5
    print("relative error", n, err, flush=True)
    assert err <= 2.5e-15
