"""The right-hand side of the factored finest level (no element inverses) against
the stored form's on the same problem, over every kind of source."""
import numpy as np
import pytest

from paper_1910_11463_amd import workloads as wl
from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu


# one element, a row and a column of elements, odd extents, more elements than a
# thread block; boxes with three different edges
@pytest.mark.parametrize("n", [(1, 1, 1), (3, 1, 7), (5, 4, 3), (9, 7, 5)])
@pytest.mark.parametrize("dual,inflow", [(None, False), ("all", False), ("each", True), (None, True)])
def test_factored_rhs_equals_stored(n, dual, inflow):
    """Both forms solve the element system in FP64; its condition number is a few
    hundred here (mass matrix 27, transport part up to kappa / sigma_t), so they
    agree to a few hundred rounding errors: 1e-12 of the largest entry."""
    need_gpu()
    from paper_1910_11463_amd.solver import Solver
    mesh = wl.hex_mesh(*n, hi=(1.0, 0.7, 1.9))
    E, N = mesh.n_elem, mesh.n_dof
    rng = np.random.default_rng(17)
    om, w = Solver.level_symmetric(4)
    M = len(w)
    st = wl.log_uniform(E, 0.1, 10.0, seed=4)
    ext = rng.uniform(-1.0, 1.0, size=(M, N) if dual == "each" else N)
    g = rng.uniform(0.0, 1.0, size=(M, N))
    out = []
    for factored in (1, 0):
        s = Solver(fine_factored=factored)
        s.set_mesh(mesh)
        s.set_quadrature(om, w)
        s.set_materials(st, 0.5 * st, np.full(E, 0.7))
        if dual:
            s.set_dual_source(ext, per_direction=dual == "each")
        if inflow:
            for m in range(M):
                s.set_inflow(g[m], m)
        out.append([s.export_fine_operator(m)[3] for m in (0, 5, 12, 23)])
        s.close()
    for a, b in zip(*out):
        assert np.abs(a - b).max() <= 1e-12 * np.abs(b).max()
