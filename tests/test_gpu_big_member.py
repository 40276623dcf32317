"""Tile sweeps of a member of more than 1 GiB per vector (64-bit places instead of
buffer instructions): one direction of a 65 x 64 x 4033 mesh against the exact sweep."""
import os

import numpy as np
import pytest

from paper_1910_11463_amd import binding as B
from paper_1910_11463_amd import workloads as wl
from tests.gpu_util import need_gpu, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile_xy", [8, 16])
def test_member_beyond_one_gib(tile_xy):
    """The inverse of the scaled operator carries an element's residual along at
    most nx + ny + nz = 4162 elements, so tol_inner = 1e-10 leaves a relative error
    below 4.2e-7: bound 1e-6."""
    need_gpu()
    from oracle import cpu_sweep as CS
    from paper_1910_11463_amd.solver import Solver
    nx, ny, nz = 65, 64, 4033
    mesh = wl.hex_mesh(nx, ny, nz, hi=(nx / 64, ny / 64, nz / 64))
    E = mesh.n_elem
    assert (E + nx + 64) * 64 > 1 << 30
    st = wl.log_uniform(E, 0.1, 10.0, seed=5)
    om, w = np.array([[0.3, -0.5, np.sqrt(0.66)]]), np.array([1.0])
    print("exact sweep of", E, "elements", flush=True)
    ref, _ = CS.sweep_all(mesh, st, 0.5 * st, np.ones(E), om, w, threads=min(16, os.cpu_count() or 1))
    print("setup and V-cycles", flush=True)
    s = Solver(tol_inner=1e-10, max_inner=100, relax_pre=b"TTT", relax_post=b"TTT", relax_pre_coarse=b"F",
               relax_post_coarse=b"", tile_xy=tile_xy, streams=1, batch_size=1, filter_r=1.0,
               allow_any_weight_sum=1)
    s.set_mesh(mesh)
    s.set_quadrature(om, w)
    s.set_materials(st, 0.5 * st, np.ones(E))
    psi, _, stats, rc = s.transport_sweep(mode=B.PAIR_BATCHED)
    s.close()
    assert rc == B.PAIR_OK
    print("V-cycles", stats["vcycles_total"], "error", rel(psi, ref), flush=True)
    assert rel(psi, ref) <= 1e-6
