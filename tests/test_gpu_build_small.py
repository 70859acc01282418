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


@pytest.mark.parametrize("n", [8193, 16384, 16385])
@pytest.mark.parametrize("grid", [(16, 16, 16), (32, 32, 32), (32, 33, 32), (33, 32, 32)])
def test_gated_limits(n, grid):
    """The builds of a Verlet list go further (16384 particles, 1024 rows of 32
    cells): the pairs within the cutoff after a rebuild, after an update that
    skips it, and after one that moves every particle."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2202_06427_amd.md as md
    rc, skin = 1.8, 0.2
    H = np.diag([0.5 * (rc + skin) * k * (1 + 1e-6) for k in grid])
    x = W.uniform_in_box(n, H, 72)
    step = W.uniform_in_box(n, np.diag([0.04] * 3), 73)
    y = W.uniform_in_box(n, H, 74)
    xt = torch.from_numpy(x).to("cuda:0")
    vl = md.VerletList(xt, H, rc, skin, lcell=2, capacity=400)
    assert vl.box.info()["grid"] == list(grid)
    F = torch.zeros((n, 3), dtype=torch.float64, device="cuda:0")
    E = torch.zeros(1, dtype=torch.float64, device="cuda:0")
    C = torch.zeros(1, dtype=torch.int64, device="cuda:0")
    for z, rebuilds in ((x, 1), (x + step, 1), (y, 2)):
        xt.copy_(torch.from_numpy(z))
        vl.update(xt)
        vl.lj(0.3, 1.0, F, E, count=C)
        assert vl.info()["rebuilds"] == rebuilds and vl.info()["overflow"] == 0
        assert int(C.item()) == oracle.compute(z, H, rc)["count"]
