"""Near thresholds beyond the cutoff and beyond the boxes of the sweep's groups:
every pair in range is then evaluated in FP64, no pair out of range and no
empty row or column is.  Against the oracle with the FP64 form's tolerances
(1e-12 of the energy's terms, 1e-11 of a particle's force magnitudes)."""
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


@pytest.mark.parametrize("near_factor", [4.0, 30.0, 1e6, 1e30])
@pytest.mark.parametrize("n", [1, 17, 33, 1500])
def test_all_pairs_near(clm, n, near_factor):
    H, rc = W.triclinic_h((31.0, 30.0, 33.0), (80.0, 95.0, 100.0)), 5.0
    sigma, eps = 0.3 * rc, 0.3
    x = W.uniform_in_box(n, H, 21)
    ref = oracle.compute(x, H, rc, lj=(sigma, eps), lj_grad=True, lj_fabs=True)
    cl = clm.CellList(torch.from_numpy(x).to("cuda:0"), clm.Box(H, rc, 2), precision="fp32")
    scale = abs(ref["lj_energy"]) + 2 * eps * ref["count"]
    e, c = cl.lj_energy(sigma, eps, near_factor=near_factor)
    assert int(c.item()) == ref["count"]
    assert abs(e.item() - ref["lj_energy"]) <= 1e-12 * scale
    out = cl.lj_forces(sigma, eps, near_factor=near_factor, half=False)
    assert int(out["count"].item()) == ref["count"]
    assert abs(out["energy"].item() - ref["lj_energy"]) <= 1e-12 * scale
    err = np.linalg.norm(out["forces"].cpu().numpy() + ref["lj_grad"], axis=1)
    assert np.all(err <= 1e-11 * ref["lj_fabs"])
