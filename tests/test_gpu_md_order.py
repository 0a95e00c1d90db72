"""The gathering molecular-dynamics kernels where their work order can go wrong:
the smallest lattice, extents that split into tiles in y with a ragged last
workgroup, and su(3) force and momentum arrays aligned to one double only."""
import pytest
import torch

import oracle as O
from oracle import md
from paper_0910_0262_amd import Lattice, synth

from ._gpu_helpers import max_rel, to_dev

pytestmark = pytest.mark.gpu
KAPPA, CSW, BETA = 0.124, 1.1, 5.6

# (20, 18, 14, 2): tiles of 9 x 14 rows (two along y), 5040 sites per parity = 78 workgroups and 48 sites
DIMS = [(2, 2, 2, 2), (2, 6, 4, 2), (20, 18, 14, 2)]


@pytest.fixture(scope="module", params=DIMS, ids=lambda d: "x".join(map(str, d)))
def case(request):
    dims = request.param
    print(f"[md order dims={dims}]", flush=True)
    u = torch.as_tensor(synth.random_su3_field(dims, 0.3, 11))
    lat = Lattice(dims, KAPPA, CSW)
    lat.load_gauge(to_dev(u))
    yield dims, lat, u
    lat.close()


# FP64 on both sides: sums of up to 6 staples or 24 leaf terms of unit-size
# matrices, a few hundred roundings of 1.1e-16 relative to the largest entry
def test_gauge_force(case):
    dims, lat, u = case
    g_ref = md.gradient(lambda v: md.gauge_action(v, BETA), u)
    s, g, f = lat.gauge_action_force(BETA)
    s_ref = float(md.gauge_action(u, BETA))
    assert abs(s - s_ref) < 1e-12 * abs(s_ref)
    assert max_rel(g, g_ref) < 1e-12
    assert max_rel(f, O.project_force(u, g_ref)) < 1e-12
    assert lat.gauge_action_force(BETA, want_G=False, want_F=False)[0] == s


def test_det_force_and_clover(case):
    dims, lat, u = case
    g_ref = md.gradient(lambda v: md.clover_det_action(v, KAPPA, CSW), u)
    _, g, f = lat.clover_det_action_force()
    assert max_rel(g, g_ref) < 1e-11
    assert max_rel(f, O.project_force(u, g_ref)) < 1e-11
    a, _ = lat.get_clover()
    blocks = O.CloverSetup(u, KAPPA, CSW).clover_blocks()  # (Lt, Lz, Ly, Lx, 2, 6, 6)
    diag = torch.diagonal(blocks, dim1=-2, dim2=-1).real.reshape(lat.V, 2, 6)
    assert float((a.cpu()[:, :, :6] - diag).abs().max()) < 1e-14


def test_one_double_alignment(case):
    """F and P whose address is 8 modulo 16 give the aligned arrays' values."""
    from paper_0910_0262_amd import capi

    dims, lat, u = case
    n = lat.V * 32
    f0 = torch.empty(n, dtype=torch.float64, device="cuda")
    f1 = torch.empty(n + 1, dtype=torch.float64, device="cuda")[1:]
    assert f1.data_ptr() % 16 == 8
    for f in (f0, f1):
        capi.qcd_gauge_action_force(lat.ctx, BETA, None, f, lat.V)
    assert torch.equal(f0, f1)
    p = to_dev(synth.momenta(dims, 3)).reshape(-1)
    p1 = torch.empty(n + 1, dtype=torch.float64, device="cuda")[1:]
    p1.copy_(p)
    ends = []
    for q in (p, p1):
        uu = to_dev(u)
        lat.md_trajectory(uu, q, None, 0.02, 2, beta=BETA, n_f=0.0)
        ends.append(uu)
    assert torch.equal(p, p1) and torch.equal(ends[0], ends[1])
    lat.load_gauge(to_dev(u))


@pytest.mark.parametrize("scale", [0.01, 0.3, 0.42, 0.44, 3.0])
def test_link_move(scale):
    """A force-free trajectory is U -> exp(i dt P) U: the power series, the closed form, and both
    sides of the line between them (c1 = 0.1875, which these momenta cross between 0.42 and 0.44)."""
    dims = (2, 6, 4, 2)
    u = torch.as_tensor(synth.random_su3_field(dims, 0.3, 5))
    p = torch.as_tensor(synth.momenta(dims, 5))
    p = p / p.norm(dim=-1, keepdim=True) * 4.0 * scale  # c1 = |h P|^2 / 4 = scale^2 with h = dt / 2 = 0.5
    lat = Lattice(dims, KAPPA, CSW)
    ud, pd = to_dev(u), to_dev(p)
    lat.md_trajectory(ud, pd, None, 1.0, 1, beta=0.0, n_f=0.0)
    ref = O.expi_su3(p, 1.0) @ u
    # two moves, each a few ten roundings of unit-size entries
    assert float((ud.cpu() - ref).abs().max()) < 2e-14
    assert torch.equal(pd.cpu(), p)
    lat.close()


def test_long_trajectory_equals_its_parts():
    """70 pure-gauge steps (more than the actions held at a time) against ten at a time."""
    dims, n = (2, 6, 4, 2), 70
    lat = Lattice(dims, KAPPA, CSW)
    ends = []
    for part in (n, 10):
        u, p, acts = to_dev(synth.random_su3_field(dims, 0.3, 6)), to_dev(synth.momenta(dims, 6)), []
        for _ in range(n // part):
            acts += lat.md_trajectory(u, p, None, 0.02, part, beta=BETA, n_f=0.0, reunitarize=True)[0]
        ends.append((u, p, torch.tensor(acts, dtype=torch.float64)))
    for a, b in zip(*ends):
        assert float((a.cpu() - b.cpu()).abs().max() / b.abs().max()) < 1e-13
    lat.close()


def test_copies_after_a_failed_trajectory():
    """A trajectory that stops with QCD_ECLOVER leaves links whose every copy agrees."""
    from paper_0910_0262_amd import QCDError

    dims = (4, 4, 4, 4)
    u, p = to_dev(synth.random_su3_field(dims, 1.0, 1)), to_dev(synth.momenta(dims, 1))
    xi = to_dev(synth.heatbath_xi(dims, 1))[None]
    lat = Lattice(dims, 0.2, 5.0)
    with pytest.raises(QCDError) as err:
        lat.md_trajectory(u, p, xi, 0.1, 1, beta=BETA, n_f=1.0, prec="mixed")
    assert err.value.status == "QCD_ECLOVER"
    moved = lat.store_gauge()
    assert float((moved - u).abs().max()) > 1e-3
    lat.set_params(0.1, 0.5)
    lat.build_clover()
    fresh = Lattice(dims, 0.1, 0.5)
    fresh.load_gauge(moved)
    b = to_dev(synth.gaussian_source(dims, 1, 0))
    bs = torch.stack([b, 2.0 * b, -b])
    for prec in ("fp64", "mixed"):
        assert torch.equal(lat.solve(b, prec=prec)[0], fresh.solve(b, prec=prec)[0])
        assert torch.equal(lat.solve_multi(bs, prec=prec)[0], fresh.solve_multi(bs, prec=prec)[0])
    lat.close()
    fresh.close()
