"""Iterations replayed from captured graphs (QCD_OPT_GRAPH) where the context changes between solves."""
import numpy as np
import pytest
import torch

from paper_0910_0262_amd import Lattice, QCDError, capi, synth

from ._gpu_helpers import to_dev

pytestmark = pytest.mark.gpu
DIMS = (4, 4, 4, 4)


@pytest.fixture
def lat():
    print(f"[graph state dims={DIMS}]", flush=True)
    lat = Lattice(DIMS, 0.12, 1.0)
    lat.load_gauge(to_dev(synth.random_su3_field(DIMS, 0.3, 2)))
    yield lat
    lat.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_option_after_a_failed_solve(lat, prec):
    """QCD_ENAN ends a solve with iterations in flight: they have run before an option destroys their graphs."""
    b = synth.gaussian_source(DIMS, 2, 0)
    bad = b.copy()
    bad[1, 2, 3, 1, 2, 1] = np.nan
    b, bad = to_dev(b), to_dev(bad)
    x0, _ = lat.solve(b, prec=prec)
    for _ in range(3):
        lat.set_option(capi.QCD_OPT_GRAPH, 1)
        assert torch.equal(lat.solve(b, prec=prec)[0], x0)
        with pytest.raises(QCDError, match="ENAN"):
            lat.solve(bad, prec=prec, pipeline_depth=16)
    lat.set_option(capi.QCD_OPT_GRAPH, 0)
    assert torch.equal(lat.solve(b, prec=prec)[0], x0)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_each_work_set_has_its_own_graphs(lat, prec):
    """qcd_solve and qcd_solve_multi with one source work on different buffers; a set that
    grows for more sources moves its own."""
    bs = to_dev(np.stack([synth.gaussian_source(DIMS, 2, k) for k in range(5)]))
    one = [lat.solve(bs[k], prec=prec)[0] for k in range(3)]
    five = lat.solve_multi(bs, prec=prec)[0]
    fresh = Lattice(DIMS, 0.12, 1.0)  # its set for several sources starts with one
    fresh.load_gauge(lat.store_gauge())
    fresh.set_option(capi.QCD_OPT_GRAPH, 1)
    for _ in range(2):
        for k in range(3):
            assert torch.equal(fresh.solve(bs[k], prec=prec)[0], one[k])
            x, st = fresh.solve_multi(bs[k:k + 1].contiguous(), prec=prec)
            assert torch.equal(x[0], one[k]) and st[0]["restarts"] == 0
        assert torch.equal(fresh.solve_multi(bs, prec=prec)[0], five)
    fresh.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_clover_form_changes_between_solves(lat, prec):
    """A built clover term has the compact form, a loaded one need not: the iterations captured
    for one read other fields than the other's."""
    b = to_dev(synth.gaussian_source(DIMS, 2, 0))
    built = lat.get_clover()[0]
    other = built.clone()
    other[:, 0, 0] += 0.4  # not 2 minus the lower spin's entry
    ref, ref_stats = [], []
    for A in (built, other):
        lat.load_clover(A)
        x, st = lat.solve(b, prec=prec)
        ref.append(x)
        ref_stats.append(st)
    assert float((ref[0] - ref[1]).abs().max()) > 1e-2
    lat.set_option(capi.QCD_OPT_GRAPH, 1)
    for k in (0, 1, 0, 1):
        lat.load_clover((built, other)[k])
        x, st = lat.solve(b, prec=prec)
        assert torch.equal(x, ref[k]), k
        assert st["iters"] == ref_stats[k]["iters"] and st["restarts"] == ref_stats[k]["restarts"]
