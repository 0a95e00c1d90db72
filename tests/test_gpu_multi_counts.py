"""Numbers of right-hand sides that fill neither a power of two nor a group of four:
each solve of a block against the same right-hand side alone."""
import pytest
import torch

from paper_0910_0262_amd import Lattice, synth

from ._gpu_helpers import max_rel, random_spinor, to_dev

pytestmark = pytest.mark.gpu

# 2^4: fewer sites than a wavefront holds; (10,6,4,6): ragged workgroups, 720 sites;
# 8^3x16: many workgroups.  n = 4, 8, 12, 16 in mixed precision run on the matrix cores
DIMS = [(2, 2, 2, 2), (10, 6, 4, 6), (8, 8, 8, 16)]
COUNTS = [2, 3, 4, 5, 7, 8, 9, 12, 13, 16]
TOL = 1e-11


@pytest.fixture(scope="module", params=DIMS, ids=lambda d: "x".join(map(str, d)))
def lat(request):
    dims = request.param
    print(f"[multi counts dims={dims}]", flush=True)
    lat = Lattice(dims, 0.12, 1.0)
    lat.load_gauge(to_dev(synth.random_su3_field(dims, 0.3, 6)))
    yield lat
    lat.close()


def _residual(lat, x, b):
    return float(torch.linalg.norm((b - lat.apply("M", x)).reshape(-1)) / torch.linalg.norm(b.reshape(-1)))


# counts in falling and rising order: one work set serves them all
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_each_source_alone(lat, prec):
    b = to_dev(random_spinor((16, lat.V), 3))
    b[1] *= 1e-3  # sources of another size that stop at another iteration
    b[2, 5:] = 0.0
    alone = [lat.solve(b[k], prec=prec, tol=TOL)[0] for k in range(16)]
    for n in COUNTS[::-1] + COUNTS:
        x, _ = lat.solve_multi(b[:n].contiguous(), prec=prec, tol=TOL)
        for k in range(n):
            # the solver's own criterion holds for |Mhat^dag (..)|; the condition is below 30
            assert _residual(lat, x[k], b[k]) < 100 * TOL, (n, k)
            assert max_rel(x[k], alone[k]) < 1e4 * TOL, (n, k)


def test_zero_source_among_others(lat):
    b = to_dev(random_spinor((5, lat.V), 4))
    b[3] = 0.0
    x, _ = lat.solve_multi(b, prec="fp64", tol=TOL)
    assert float(x[3].abs().max()) == 0.0
    assert _residual(lat, x[4], b[4]) < 100 * TOL
