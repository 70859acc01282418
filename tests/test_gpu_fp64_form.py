"""The FP64 form decides every pair in FP64: no map of it re-evaluates a pair
that FP32 left open (the counters of clm_celllist_info stay at zero), and its
integers are the oracle's, also with pairs at the cutoff and at bin edges to
the last bits (distances of a lattice with steps of an eighth; the cutoff and
the edges are among them)."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def clm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2202_06427_amd as clm
    return clm


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def sets(name):
    if name == "lattice":
        H = np.diag([16.0, 16.0, 16.0])
        g = W.rng(2)
        return g.integers(0, 128, size=(4000, 3)) / 8.0, H, 3.0
    H = W.triclinic_h((31.0, 30.0, 33.0), (80.0, 95.0, 100.0))
    return W.uniform_in_box(6000, H, 3), H, 5.0


@pytest.mark.parametrize("name", ["lattice", "uniform"])
def test_no_re_evaluations(clm, name):
    x, H, rc = sets(name)
    nbins = 24
    ref = oracle.compute(x, H, rc, hist=(nbins, rc), nl=True)
    cl = clm.CellList(T(x), clm.Box(H, rc, 2), precision="fp64")

    def clean():
        i = cl.info()
        return i["guard_retests"] == 0 and i["near_evaluations"] == 0

    assert int(cl.count().item()) == ref["count"] and clean()
    h, c = cl.histogram(nbins)
    assert np.array_equal(h.cpu().numpy().astype(np.uint64), ref["hist"]) and int(c.item()) == ref["count"]
    assert clean()
    for ordered in (True, False):
        p, _ = cl.neighbor_list(sorted=ordered)
        p = p.cpu().numpy()
        p = p[np.lexsort((p[:, 1], p[:, 0]))]
        assert np.array_equal(p[:, 0], ref["nl_i"]) and np.array_equal(p[:, 1], ref["nl_j"])
        assert clean()
    assert int(cl.sum_d()[1].item()) == ref["count"] and clean()


@pytest.mark.parametrize("nbins", [1, 7, 24, 1000])
@pytest.mark.parametrize("top", [0.25, 1.0, 1.5])
def test_bins(clm, nbins, top):
    for name in ("lattice", "uniform"):
        x, H, rc = sets(name)
        ref = oracle.compute(x, H, rc, hist=(nbins, top * rc))
        h, _ = clm.CellList(T(x), clm.Box(H, rc, 2), precision="fp64").histogram(nbins, top * rc)
        assert np.array_equal(h.cpu().numpy().astype(np.uint64), ref["hist"]), name
