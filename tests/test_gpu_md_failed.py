"""What molecular-dynamics calls that stop with an error hand out of the work before it."""
import ctypes

import numpy as np
import pytest
import torch

import oracle as O
from paper_0910_0262_amd import Lattice, capi, synth

from ._gpu_helpers import to_dev

pytestmark = pytest.mark.gpu
DIMS, BETA, DT = (2, 2, 4, 2), 5.6, 0.02


def _trajectory(lat, u, p, xi, n):
    """(status, actions [n][3] with -1 where nothing was written) of a two-flavour trajectory in place on u, p."""
    md = capi.make_md_params(DT, n, BETA, 2.0, True, False)
    par = capi.make_params(tol=1e-11)
    acts = (ctypes.c_double * (3 * n))(*[-1.0] * (3 * n))
    ptr = [ctypes.c_void_p(t.data_ptr()) for t in (u, p, xi)]
    rc = capi.lib().qcd_md_trajectory(lat.ctx, ctypes.byref(md), *ptr, ctypes.byref(par), acts, None)
    return rc, np.array(acts).reshape(n, 3)


# the actions wait on the GPU's side for 64 steps at a time
@pytest.mark.parametrize("stop,n", [(0, 2), (1, 2), (3, 5), (63, 64), (64, 66), (66, 68)])
def test_actions_of_the_steps_before_a_failure(stop, n):
    print(f"[failed trajectory stop={stop} n={n}]", flush=True)
    u0, p0 = to_dev(synth.random_su3_field(DIMS, 0.3, 4)), to_dev(synth.momenta(DIMS, 4))
    xi = to_dev(np.stack([synth.heatbath_xi(DIMS, 4 + k) for k in range(n)]))
    lat = Lattice(DIMS, 0.12, 1.0)
    u, p = u0.clone(), p0.clone()
    expect = np.full((n, 3), -1.0)
    if stop > 0:
        rc, expect[:stop] = _trajectory(lat, u, p, xi[:stop].contiguous(), stop)
        assert rc == capi.QCD_OK
    xi[stop, 3, 1, 1] = float("nan")
    v, q = u0.clone(), p0.clone()
    rc, acts = _trajectory(lat, v, q, xi, n)
    assert rc == capi.QCD_ENAN
    assert np.array_equal(acts, expect)
    assert torch.equal(p, q)
    lat.close()


def test_action_of_a_step_that_ends_beyond_the_clover_term():
    """The links of U = 1 grow rougher along the step: the clover term can be inverted where the
    force is taken, and no longer where the step ends."""
    dims, kappa, dt = (4, 4, 4, 4), 0.1, 1e-4
    p0 = torch.as_tensor(synth.momenta(dims, 9)) * (0.2 / dt)  # |dt F| is far below |P|
    u0 = torch.as_tensor(synth.unit_gauge(dims))

    def lowest(c):  # of (A - 1) / c_sw on odd sites
        a = O.CloverSetup(O.expi_su3(p0, c * dt) @ u0, kappa, 1.0).A_o
        return float(torch.linalg.eigvalsh(a).min()) - 1.0

    mid, end = lowest(0.5), lowest(1.0)
    assert 1.3 * mid > end  # both negative
    csw = 1.0 / (mid * end) ** 0.5
    lat = Lattice(dims, kappa, csw)
    u, p, s = to_dev(u0), to_dev(p0), ctypes.c_double(-1.0)
    xi, par = to_dev(synth.heatbath_xi(dims, 9)), capi.make_params(tol=1e-11)
    rc = capi.lib().qcd_hmd_step(lat.ctx, dt, *[ctypes.c_void_p(t.data_ptr()) for t in (u, p, xi)],
                                 ctypes.byref(par), ctypes.byref(s), None)
    assert rc == capi.QCD_ECLOVER
    # the links moved to the end; phi = Mhat^dag xi at U = 1, the action at the middle
    phi = O.CloverSetup(u0, kappa, csw).Mhat_dag(torch.as_tensor(synth.heatbath_xi(dims, 9)))
    mid_links = O.expi_su3(p0, 0.5 * dt) @ u0
    ref = O.action_and_gradient(mid_links, kappa, csw, phi, tol=1e-13)[0]
    assert abs(s.value - ref) < 1e-9 * abs(ref)
    lat.close()


def test_actions_left_out_are_plus_zero():
    u, p = to_dev(synth.random_su3_field(DIMS, 0.3, 4)), to_dev(synth.momenta(DIMS, 4))
    lat = Lattice(DIMS, 0.12, 1.0)
    acts, _ = lat.md_trajectory(u, p, None, DT, 2, beta=BETA, n_f=0.0)
    assert [str(a[k]) for a in acts for k in (0, 2)] == ["0.0"] * 4
    acts, _ = lat.md_trajectory(u, p, to_dev(synth.heatbath_xi(DIMS, 4))[None], DT, 1, n_f=2.0, clover_det=False)
    assert [str(a) for a in acts[0][1:]] == ["0.0"] * 2
    lat.close()
