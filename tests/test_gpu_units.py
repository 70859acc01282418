"""Sums, energies and forces do not depend on the unit of length: the same
configuration with every length multiplied by a power of two.  Wrapping, cells
and the maps are then the same operations on scaled numbers, so counts are
equal and sums scale bit for bit (forces: sums over lanes in LDS, one rounding
of the largest)."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu
H3, RC = W.triclinic_h((31.0, 30.0, 33.0), (80.0, 95.0, 100.0)), 5.0


@pytest.fixture(scope="module")
def clm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2202_06427_amd as clm
    return clm


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def lists(clm, k, precision):
    s = 2.0 ** k
    x = W.uniform_in_box(3000, H3, 12)
    return s, clm.CellList(T(s * x), clm.Box(s * H3, s * RC, 2), precision=precision)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("k", [-120, -45, 45, 120])
def test_sums(clm, k, precision):
    w = T(0.5 + W.rng(9).random(3000))
    _, a = lists(clm, 0, precision)
    s, b = lists(clm, k, precision)
    for name, args, power in (("sum_d", (), 1), ("sum_inv_d", (), -1), ("sum_w_inv_d", (w,), -1)):
        (ea, ca), (eb, cb) = getattr(a, name)(*args), getattr(b, name)(*args)
        assert int(ca.item()) == int(cb.item()), name
        assert eb.item() == ea.item() * s ** power, name


@pytest.mark.parametrize("k", [-120, -45, 45, 120])
def test_lennard_jones(clm, k):
    _, a = lists(clm, 0, "fp32")
    s, b = lists(clm, k, "fp32")
    (ea, ca), (eb, cb) = a.lj_energy(2.0, 0.3), b.lj_energy(2.0 * s, 0.3)
    assert int(ca.item()) == int(cb.item()) and ea.item() == eb.item()
    fa = a.lj_forces(2.0, 0.3, half=False, virial=True)
    fb = b.lj_forces(2.0 * s, 0.3, half=False, virial=True)
    assert int(fa["count"].item()) == int(fb["count"].item())
    for name, power in (("forces", -1), ("virial", 0), ("grad_box", -1)):
        u, v = fa[name], fb[name] * s ** -power
        assert float((u - v).abs().max()) <= 1e-14 * float(u.abs().max()), name


@pytest.mark.parametrize("ratio", [1e-40, 1e-12, 1e-9, 1e-3, 1e3, 1e9, 1e12, 1e40])
def test_sigma_far_from_the_cutoff(clm, ratio):
    """sigma from far below to far above the cutoff: the FP64 form's count, and its
    energy and forces within the FP32 form's 1e-5 (all of the same sign there)."""
    x = W.uniform_in_box(3000, H3, 12)
    sigma = ratio * RC
    out = {}
    for p in ("fp32", "fp64"):
        cl = clm.CellList(T(x), clm.Box(H3, RC, 2), precision=p)
        e, c = cl.lj_energy(sigma, 0.3)
        f = cl.lj_forces(sigma, 0.3, half=False)
        out[p] = [int(c.item()), int(f["count"].item()), e.item(), f["energy"].item(), f["forces"]]
    a, b = out["fp32"], out["fp64"]
    assert a[:2] == b[:2]
    if 1e-3 <= ratio <= 1e3:
        assert abs(a[2] - b[2]) <= 1e-5 * abs(b[2]) and abs(a[3] - b[3]) <= 1e-5 * abs(b[3])
        assert float((a[4] - b[4]).abs().max()) <= 1e-5 * float(b[4].abs().max())
