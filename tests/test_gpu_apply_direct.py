"""Operators on the caller's own arrays: every form of qcd_apply against the
one-work-item form on packed fields, and arrays that share memory."""
import numpy as np
import pytest
import torch

from paper_0910_0262_amd import Lattice, capi, synth

from ._gpu_helpers import max_rel, random_spinor, to_dev

pytestmark = pytest.mark.gpu

# (2,2,2,2): 8 sites per parity; (10,6,4,6): a ragged last workgroup; (32,32,32,4): the
# largest lattice that takes the caller's arrays on both sides; (32,32,34,4): the next one
DIMS = [(2, 2, 2, 2), (10, 6, 4, 6), (32, 32, 32, 4), (32, 32, 34, 4)]
OPS = ["M", "Mdag", "Mhat", "Mhatdag", "MdagM"]


@pytest.fixture(scope="module", params=DIMS, ids=lambda d: "x".join(map(str, d)))
def lat(request):
    dims = request.param
    print(f"[apply direct dims={dims}]", flush=True)
    lat = Lattice(dims, 0.124, 1.0)
    lat.load_gauge(to_dev(synth.random_su3_field(dims, 0.3, 2)))
    yield lat
    lat.close()


@pytest.mark.parametrize("recon", [12, 18])
@pytest.mark.parametrize("op", OPS)
def test_forms_agree(lat, op, recon):
    n = lat.V if op in ("M", "Mdag") else lat.Vh
    psi = to_dev(random_spinor((n,), 7))
    lat.set_option(capi.QCD_OPT_LINK_RECON, recon)
    out = lat.apply(op, psi)
    lat.set_option(capi.QCD_OPT_SMALL_GRID, 0)
    ref = lat.apply(op, psi)
    lat.set_option(capi.QCD_OPT_SMALL_GRID, 2)
    lat.set_option(capi.QCD_OPT_LINK_RECON, 12)
    # the same sums in another order: up to four stencils of some 100 roundings each
    assert max_rel(out, ref) < 1e-13


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("op", OPS)
def test_arrays_that_share_memory(lat, op, prec):
    """The result laid over part of the input is the result laid elsewhere."""
    full = op in ("M", "Mdag")
    if full and prec == "mixed":
        pytest.skip("the full-lattice operators are FP64 only")
    n = lat.V if full else lat.Vh
    code = {"M": 0, "Mdag": 1, "Mhat": 2, "Mhatdag": 3, "MdagM": 4}[op]
    psi = to_dev(random_spinor((n,), 8))
    ref = lat.apply(op, psi, prec)
    for shift in (1, n // 2):
        buf = torch.zeros((n + shift, 4, 3), dtype=torch.complex128, device="cuda")
        buf[:n] = psi
        src, dst = buf[:n], buf[shift:]
        capi.qcd_apply(lat.ctx, code, {"fp64": 0, "mixed": 1}[prec], src, dst, n)
        torch.cuda.synchronize()
        assert max_rel(dst, ref) < 1e-13
    assert np.isfinite(float(ref.abs().max()))
