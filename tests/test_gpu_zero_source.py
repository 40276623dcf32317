"""Zero right-hand sides: x = 0 without a single V-cycle, for every way in which a
sweep's source can be zero; nonzero ones in the same problem still solved."""
import ctypes

import numpy as np
import pytest

from tests.gpu_util import need_gpu, solver_for

pytestmark = pytest.mark.gpu


def _cycles(call):
    """The call's result and the finest-level half-sweeps it launched."""
    from paper_1910_11463_amd import binding as B
    B.check(B.pair_profile_enable(1))
    out = call()
    k, ms, by = ctypes.c_int64(), ctypes.c_double(), ctypes.c_double()
    B.check(B.pair_profile_read(0, ctypes.byref(k), ctypes.byref(ms), ctypes.byref(by)))
    B.check(B.pair_profile_enable(0))
    return out, k.value


@pytest.mark.parametrize("cfg", [2, 3])
@pytest.mark.parametrize("mode,streams", [("plain", 1), ("batched", 1), ("batched", 2)])
@pytest.mark.parametrize("source", ["none", "ext", "ext_per_direction", "inflow_one_direction"])
def test_zero_sweep_launches_no_cycle(cfg, mode, streams, source):
    need_gpu()
    from paper_1910_11463_amd import binding as B
    from paper_1910_11463_amd import workloads as wl
    mode = B.PAIR_PLAIN if mode == "plain" else B.PAIR_BATCHED
    w = wl.make_config(cfg, scale=3)
    s = solver_for(w, 2, use_graph=0, streams=streams, batch_size=4, keep_hierarchy=1)
    zero = np.zeros(s.N)
    s.set_materials(w.mats.sigma_t, w.mats.sigma_s, np.zeros(s.E))
    if source == "ext":
        s.set_dual_source(zero)
    elif source == "ext_per_direction":
        s.set_dual_source(np.zeros((s.M, s.N)), per_direction=True)
    elif source == "inflow_one_direction":
        s.set_inflow(np.ones(s.N), m=0)
    for phi_in in (None, zero):
        (psi, phi, st, rc), k = _cycles(lambda: s.transport_sweep(mode=mode, phi_in=phi_in))
        assert rc == B.PAIR_OK
        one = source == "inflow_one_direction"
        assert not psi[1:].any() and psi[0].any() == one and phi.any() == one
        assert st["vcycles_total"] == st["vcycles_max"] and (k > 0) == one
    # the same problem with a source again
    s.set_materials(w.mats.sigma_t, w.mats.sigma_s, w.mats.q)
    (psi, phi, st, rc), k = _cycles(lambda: s.transport_sweep(mode=mode))
    assert rc == B.PAIR_OK and k > 0 and phi.any()
    s.close()


def test_zero_gradient_launches_no_cycle():
    need_gpu()
    from paper_1910_11463_amd import binding as B
    from paper_1910_11463_amd import workloads as wl
    w = wl.make_config(2, scale=3)
    s = solver_for(w, 2, use_graph=0, keep_hierarchy=1)
    assert s.solve(mode=B.PAIR_BATCHED)[3] == B.PAIR_OK
    (gt, gs, pa, st, rc), k = _cycles(lambda: s.adjoint(np.zeros(s.N), mode=B.PAIR_BATCHED))
    assert rc == B.PAIR_OK and k == 0 and not gt.any() and not gs.any() and not pa.any()
    (gt, gs, pa, st, rc), k = _cycles(lambda: s.adjoint(np.ones(s.N), mode=B.PAIR_BATCHED))
    assert rc == B.PAIR_OK and k > 0 and gs.any()
    s.close()
