"""The clover term built from links against the same term loaded: both forms of
the building kernel and everything that is derived from A."""
import pytest
import torch

from paper_0910_0262_amd import Lattice, capi, synth

from ._gpu_helpers import max_rel, random_spinor, to_dev

pytestmark = pytest.mark.gpu

# (2,2,2,2): 8 sites per parity; (10,6,4,6): a ragged last workgroup; (16,16,16,8): the
# last size of the form with six wavefronts; (18,14,14,10), (16,16,16,10): the other
# form, with and without a ragged last workgroup
DIMS = [(2, 2, 2, 2), (10, 6, 4, 6), (16, 16, 16, 8), (18, 14, 14, 10), (16, 16, 16, 10)]


@pytest.fixture(scope="module", params=DIMS, ids=lambda d: "x".join(map(str, d)))
def pair(request):
    dims = request.param
    print(f"[clover build dims={dims}]", flush=True)
    u = to_dev(synth.random_su3_field(dims, 0.3, 4))
    built, loaded = Lattice(dims, 0.124, 1.2), Lattice(dims, 0.124, 1.2)
    built.load_gauge(u)
    loaded.load_gauge(u, build_clover=False)
    loaded.load_clover(built.get_clover()[0])
    yield built, loaded
    built.close()
    loaded.close()


def test_blocks_and_determinant(pair):
    built, loaded = pair
    a, ai = built.get_clover()
    b, bi = loaded.get_clover()
    assert torch.equal(a, b)
    # the same elimination on the same values: a few hundred roundings at a condition below 10
    assert max_rel(ai, bi) < 1e-13
    s, t = (x.clover_det_action_force(False, False)[0] for x in pair)
    # twelve logarithms per site, 1e-16 each
    assert abs(float(s) - float(t)) < 1e-14 * built.V


@pytest.mark.parametrize("compact", [0, 1])
@pytest.mark.parametrize("bits", [16, 32])
def test_operators(pair, bits, compact):
    psi = to_dev(random_spinor((pair[0].Vh,), 5))
    out = {}
    for prec in ("fp64", "mixed"):
        for x in pair:
            # with the term already there: the FP32 copies are made for it now
            x.set_option(capi.QCD_OPT_COMPACT_CLOVER, compact)
            x.set_option(capi.QCD_OPT_MIXED_CLOVER, bits)
        out[prec] = [x.apply("Mhat", psi, prec) for x in pair]
        for x in pair:
            x.set_option(capi.QCD_OPT_MIXED_CLOVER, 16)
            x.set_option(capi.QCD_OPT_COMPACT_CLOVER, 1)
    assert max_rel(*out["fp64"]) < 1e-13
    # a value next to a rounding boundary may fall to either side: units of 2^-11 of a
    # site's or block's scale, a few of them; against FP64 all of them, 24 terms a row
    assert max_rel(*out["mixed"]) < 2.0 ** -8
    assert max_rel(out["mixed"][0], out["fp64"][0]) < 24 * 2.0 ** -11
