"""The force gather in sparse boxes (a wave takes a whole tile of a particle or
two, and of full tiles where there are clumps) against the oracle, with wrapped
particles, images and the virial: forces within 1e-5 / 1e-11 of a particle's
force magnitudes, energy within 1e-6 / 1e-12 of its terms, tensors of the sum of
the magnitudes times the cutoff (four boxes for the box gradient)."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu
BOXES = {
    "3d": (W.triclinic_h((60.0, 58.0, 63.0), (85.0, 95.0, 98.0)), 1.0, 12000),
    "3d_few": (np.diag([40.0, 40.0, 40.0]), 1.0, 4400),      # at the number of tiles that chooses
    "2d": (np.array([[400.0, 30.0], [0.0, 380.0]]), 1.5, 12000),
}


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("name", list(BOXES))
def test_sparse_forces(name, precision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2202_06427_amd as clm
    H, rc, n = BOXES[name]
    dim = H.shape[0]
    x = W.uniform_in_box(n, H, 81)
    clump = H @ np.full(dim, 0.5) + W.rng(82).normal(scale=1.5 * rc, size=(700, dim))
    x = np.concatenate([x, clump])
    x[::3] += H @ (np.arange(dim) * 2.0 - 1.0)
    sigma, eps = 0.3 * rc, 0.3
    ref = oracle.compute(x, H, rc, lj=(sigma, eps), lj_grad=True, lj_fabs=True)
    cl = clm.CellList(torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0"), clm.Box(H, rc, 2), precision=precision)
    tol_e, tol_f = (1e-6, 1e-5) if precision == "fp32" else (1e-12, 1e-11)
    top = ref["lj_fabs"].sum()
    for virial in (False, True):
        out = cl.lj_forces(sigma, eps, virial=virial, half=False)
        assert int(out["count"].item()) == ref["count"]
        assert abs(out["energy"].item() - ref["lj_energy"]) <= tol_e * (abs(ref["lj_energy"]) + 2 * eps * ref["count"])
        err = np.linalg.norm(out["forces"].cpu().numpy() + ref["lj_grad"], axis=1)
        assert np.all(err <= tol_f * ref["lj_fabs"])
        assert np.abs(out["grad_box"].cpu().numpy() - ref["dEdH"]).max() <= tol_f * 4 * top
        if virial:
            assert np.abs(out["virial"].cpu().numpy() - ref["virial"]).max() <= tol_f * rc * top
        again = cl.lj_forces(sigma, eps, virial=virial, half=False)
        assert torch.equal(out["forces"], again["forces"]) and torch.equal(out["energy"], again["energy"])
