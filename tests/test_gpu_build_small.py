"""Builds on both sides of the limits of the one-launch binning (8192 particles)
and the one-launch tiles (256 rows of 32 cells): every pair of the oracle, from
the list and from the count (the tiles hold every particle once)."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [700, 8191, 8192, 8193])
@pytest.mark.parametrize("grid", [(16, 16, 16), (16, 15, 17), (32, 16, 16), (33, 16, 16), (32, 17, 16), (32, 256), (32, 257)])
def test_limits(n, grid):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2202_06427_amd as clm
    rc = 2.0
    H = np.diag([0.5 * rc * k * (1 + 1e-6) for k in grid])
    x = W.uniform_in_box(n, H, 71)
    box = clm.Box(H, rc, 2)
    assert box.info()["grid"] == list(grid)
    cl = clm.CellList(torch.from_numpy(x).to("cuda:0"), box)
    ref = oracle.compute(x, H, rc, nl=True)
    for _ in range(2):
        p = cl.neighbor_list(distances=False, sorted=True)[0].cpu().numpy()
        assert np.array_equal(p[:, 0], ref["nl_i"]) and np.array_equal(p[:, 1], ref["nl_j"])
        assert int(cl.count().item()) == ref["count"]
        cl.build(torch.from_numpy(x).to("cuda:0"))
