"""Verlet lists of 400000 particles and more: lists built anew from the same
positions give the same bits of forces, energy and virial (cells of a few
particles, whose order a build fixes; the order within a list does not depend on
the order in which waves run)."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [400_000, 450_001])
def test_lists_are_reproducible(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2202_06427_amd.md as md
    H = np.diag([(n / 0.1) ** (1.0 / 3.0)] * 3)
    x = torch.from_numpy(W.uniform_in_box(n, H, 5)).to("cuda:0")
    got = []
    for _ in range(3):
        vl = md.VerletList(x, H, 5.0, 0.8, lcell=2, capacity=200)
        F = torch.empty((n, 3), dtype=torch.float64, device="cuda:0")
        E = torch.zeros(1, dtype=torch.float64, device="cuda:0")
        V = torch.zeros((3, 3), dtype=torch.float64, device="cuda:0")
        vl.update(x)
        vl.lj(1.5, 0.3, F, E, virial=V)
        assert vl.info()["overflow"] == 0
        got.append((F, E, V))
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert torch.equal(a, b)
