"""The Verlet list's shared lists of four rows where their grouping can go wrong:
one to a few groups, tiles of a particle or two beside full ones, 2D, cells of
many particles, coincident coordinates along an axis; a list whose order must
not vary.  Against the FP64 force map of the same positions: the same pairs,
sums of the same FP64 terms in another order (1e-12 of the largest sum of
pair-force magnitudes bounds it; at most 400 terms a particle, each off by a
few 2^-53)."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def md():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2202_06427_amd.md as md
    return md


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def points(name, n):
    r = W.rng(60 + n)
    if name == "2d":
        H = np.array([[60.0, 7.0], [0.0, 55.0]])
        return W.uniform_in_box(n, H, 61 + n), H, 4.0
    H = np.diag([40.0, 38.0, 41.0])
    x = W.uniform_in_box(n, H, 62 + n)
    if name == "sparse":   # 10^4 cells and more, clumps of full tiles
        H = np.diag([60.0, 60.0, 60.0])
        return np.concatenate([W.uniform_in_box(8 * n, H, 63), 20.0 + r.normal(scale=1.5, size=(n // 4, 3))]), H, 1.2
    if name == "plane":    # one z, few values of y
        x[:, 2] = 20.0
        x[:, 1] = np.round(x[:, 1] / 2.0) * 2.0
    return x, H, 4.0


@pytest.mark.parametrize("name", ["uniform", "2d", "sparse", "plane"])
@pytest.mark.parametrize("n", [1, 3, 5, 17, 65, 2000])
def test_groups_of_rows(md, name, n):
    import paper_2202_06427_amd as clm
    x, H, rc = points(name, n)
    n, dim, sig, eps = len(x), H.shape[0], 0.35 * rc, 0.3
    xd = T(x)
    vl = md.VerletList(xd, H, rc, 0.2 * rc, lcell=2, capacity=1000)
    F = torch.empty((n, dim), dtype=torch.float64, device="cuda:0")
    E = torch.zeros(1, dtype=torch.float64, device="cuda:0")
    V = torch.zeros((dim, dim), dtype=torch.float64, device="cuda:0")
    C = torch.zeros(1, dtype=torch.int64, device="cuda:0")
    vl.update(xd)
    vl.lj(sig, eps, F, E, virial=V, count=C)
    assert vl.info()["overflow"] == 0
    ref = clm.CellList(xd, clm.Box(H, rc, 2), precision="fp64").lj_forces(sig, eps, virial=True)
    assert int(C.item()) == int(ref["count"].item())
    scale = max(float(ref["forces"].abs().max()), 1e-300)
    for got, want, s in ((F, ref["forces"], scale), (V, ref["virial"], scale * rc * n)):
        assert float((got - want).abs().max()) <= 1e-11 * s
    assert abs(E.item() - ref["energy"].item()) <= 1e-11 * max(abs(ref["energy"].item()), eps * max(int(C.item()), 1))
