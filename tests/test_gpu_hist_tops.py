"""Distance histograms whose top is far below, at and far above the cutoff:
exact counts, and exact sums of relative speeds (every second particle moves at
1 along x, so they are whole numbers)."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("top", [1e-8, 1e-6, 1.0, 1e6, 1e12, 1e19, 1e20, 1e21, 1e22, 1e25, 1e100])
def test_tops(top, precision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2202_06427_amd as clm
    H, rc, nbins = W.triclinic_h((31.0, 30.0, 33.0), (80.0, 95.0, 100.0)), 5.0, 10
    x = W.uniform_in_box(2000, H, 5)
    v = np.zeros((2000, 3))
    v[::2, 0] = 1.0
    ref = oracle.compute(x, H, rc, hist=(nbins, top * rc), vel_x=v, dist_vel_hist=(nbins, top * rc))
    T = lambda a: torch.from_numpy(a).to("cuda:0")
    cl = clm.CellList(T(x), clm.Box(H, rc, 2), precision=precision)
    h, c = cl.histogram(nbins, top * rc)
    assert int(c.item()) == ref["count"]
    assert np.array_equal(h.cpu().numpy().astype(np.uint64), ref["hist"])
    h, s, c = cl.dist_vel_histogram(T(v), nbins, top * rc)
    assert int(c.item()) == ref["count"]
    assert np.array_equal(h.cpu().numpy().astype(np.uint64), ref["dv_hist"])
    assert np.array_equal(s.cpu().numpy(), ref["dv_sum"])
