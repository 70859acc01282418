"""A Verlet list that has never been updated is an empty list: zero forces,
energy, virial and pairs, velocities as they were, and their kinetic energy."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("kick", [False, True])
def test_no_update_yet(dim, kick):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2202_06427_amd.md as md
    n, H = 3000, np.diag([40.0] * dim)
    x = torch.from_numpy(W.uniform_in_box(n, H, 5)).to("cuda:0")
    v = torch.from_numpy(W.rng(6).normal(size=(n, dim))).to("cuda:0")
    v0 = v.clone()
    one = lambda: torch.full((1,), 7.0, dtype=torch.float64, device="cuda:0")
    F = torch.full((n, dim), 7.0, dtype=torch.float64, device="cuda:0")
    E, K, V = one(), one(), torch.full((dim, dim), 7.0, dtype=torch.float64, device="cuda:0")
    C = torch.full((1,), 7, dtype=torch.int64, device="cuda:0")
    vl = md.VerletList(x, H, 4.0, 0.8, lcell=2, capacity=200)
    it = md.Integrator(n, dim, 2.0, 0.001, x.device) if kick else None
    vl.lj(1.5, 0.3, F, E, virial=V, count=C, integrator=it, v=v if kick else None, ke=K if kick else None)
    assert float(F.abs().max()) == 0.0 and float(E.abs()) == 0.0 and float(V.abs().max()) == 0.0 and int(C.item()) == 0
    assert torch.equal(v, v0)
    if kick:  # sum of n dim squares in FP64
        want = float((v0 * v0).sum())
        assert abs(K.item() - want) <= 1e-12 * want
    vl.update(x)
    vl.lj(1.5, 0.3, F, E, virial=V, count=C)
    assert int(C.item()) > 0 and float(F.abs().max()) > 0.0
