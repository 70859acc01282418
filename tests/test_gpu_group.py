"""GPU parity of the group sweep (16 particles against 16 candidates at a time)
against the CPU oracle at the sizes where its tiling can go wrong: groups,
tiles and candidate blocks that are full, one short and one over, boxes with
the fewest cells a row may have, long thin rows, one particle, two sets of
very different sizes, a smaller map cutoff, histograms of few and many bins
that end below, at and above the cutoff, and values that sit at zero.

Counts and histograms are exact.  Sums of FP32 terms (each off by at most
about 10 u, u = 2^-24, and summed in runs of at most 5) are within 2e-6 of
the sum of their magnitudes.  A speed |v_j - v_i| of FP32 velocities is also
off by the rounding of the velocities themselves, at most 2 u max|v| sqrt(dim)
a pair whatever the speed is."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu
TOL = {"fp32": 2e-6, "fp64": 1e-12}


@pytest.fixture(scope="module")
def clm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2202_06427_amd as clm
    return clm


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


TRI3 = W.triclinic_h((31.0, 30.0, 33.0), (80.0, 95.0, 100.0))
TRI2 = np.array([[55.0, -12.0], [0.0, 50.0]])
# name -> (box, cutoff, lcell, lcell_x)
BOXES = {
    "tri3": (TRI3, 5.0, 2, None),
    "fewest3": (np.diag([30.0, 30.0, 30.0]), 11.5, 2, None),   # five cells on an axis
    "row3": (np.diag([200.0, 9.1, 9.1]), 3.0, 1, 4),           # long rows, three cells across
    "tri2": (TRI2, 6.0, 2, None),
    "l1_2": (np.diag([40.0, 40.0]), 13.0, 1, None),            # three cells on an axis
}


def check(clm, x, H, rc, lcell, lcell_x, precision, y=None, cutoff=None, nbins=17, hi=None):
    dim = H.shape[0]
    rm = rc if cutoff is None else cutoff
    hi = rm if hi is None else hi
    v = W.rng(7).normal(size=x.shape)
    vy = None if y is None else W.rng(8).normal(size=y.shape)
    w = 0.5 + W.rng(9).random(len(x))
    wy = None if y is None else 0.5 + W.rng(10).random(len(y))
    ref = oracle.compute(x, H, rm, y, sum_d=True, sum_inv_d=True, lj=(0.4 * rc, 0.3), hist=(nbins, hi),
                         rel_hist=(nbins, 3.0), vel_x=v, vel_y=vy, weights=(w, wy),
                         dist_vel_hist=(nbins, hi))
    cl = clm.CellList(T(x), clm.Box(H, rc, lcell, lcell_x=lcell_x), y=None if y is None else T(y),
                      precision=precision)
    assert not cl.box.info()["small_box"]
    tol = TOL[precision]
    kw = {"cutoff": cutoff}
    vmax = max(np.abs(v).max(), 0.0 if vy is None else np.abs(vy).max())
    pair = 0.0 if precision == "fp64" else 2 * 2.0 ** -24 * vmax * np.sqrt(dim)  # speed error of one pair
    tv, tvy, tw, twy = T(v), None if y is None else T(vy), T(w), None if y is None else T(wy)
    assert int(cl.count(**kw).item()) == ref["count"]
    h, c = cl.histogram(nbins, hi, **kw)
    assert int(c.item()) == ref["count"]
    assert np.array_equal(h.cpu().numpy().astype(np.uint64), ref["hist"])
    for got, want in ((cl.sum_d(**kw), ref["sum_d"]), (cl.sum_inv_d(**kw), ref["sum_inv_d"]),
                      (cl.sum_w_inv_d(tw, twy, **kw), ref["sum_w_inv_d"])):
        assert int(got[1].item()) == ref["count"]
        if np.isfinite(want):
            assert abs(got[0].item() - want) <= tol * abs(want)
        else:  # coincident particles: 1/d is infinite (the oracle's compensated sum says NaN)
            assert got[0].item() == np.inf
    if y is None:
        e, c = cl.lj_energy(0.4 * rc, 0.3, **kw)
        assert int(c.item()) == ref["count"]
        # every pair's terms: 4 eps (a^2 + a), a = (s/d)^6, bounded through u + 2 * 4 eps a
        assert not np.isfinite(ref["lj_energy"]) or abs(e.item() - ref["lj_energy"]) <= 10 * tol * (abs(ref["lj_energy"]) + 8 * 0.3 * ref["count"])
    h, s, c = cl.dist_vel_histogram(tv, nbins, hi, vy=tvy, **kw)
    assert int(c.item()) == ref["count"]
    assert np.array_equal(h.cpu().numpy().astype(np.uint64), ref["dv_hist"])
    assert np.allclose(s.cpu().numpy(), ref["dv_sum"], rtol=tol, atol=pair * ref["dv_hist"][:-1])
    h, s, c = cl.relspeed_histogram(tv, nbins, 3.0, vy=tvy, **kw)
    assert int(c.item()) == ref["count"]
    assert np.array_equal(h.cpu().numpy().astype(np.uint64), ref["rel_hist"])
    assert np.allclose(s.cpu().numpy(), ref["rel_sum"], rtol=tol, atol=pair * ref["rel_hist"][:-1])


@pytest.mark.parametrize("box", list(BOXES))
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 33, 64, 65, 129, 1000, 4001])
def test_sizes(clm, box, n):
    H, rc, l, lx = BOXES[box]
    x = W.uniform_in_box(n, H, 900 + n) + H @ np.full(H.shape[0], 3.0)
    check(clm, x, H, rc, l, lx, "fp32")
    check(clm, x, H, rc, l, lx, "fp64")


@pytest.mark.parametrize("nx,ny", [(1, 1), (1, 3000), (17, 3000), (700, 20), (2000, 1999)])
def test_two_sets(clm, nx, ny):
    H, rc, l, lx = BOXES["tri3"]
    check(clm, W.uniform_in_box(nx, H, 31), H, rc, l, lx, "fp32", y=W.uniform_in_box(ny, H, 32))


@pytest.mark.parametrize("nbins", [1, 2, 63, 64, 65, 1000])
@pytest.mark.parametrize("top", [1e-3, 0.3, 1.0, 1.7])
def test_bins(clm, nbins, top):
    H, rc, l, lx = BOXES["tri3"]
    x = W.uniform_in_box(3000, H, 41)
    check(clm, x, H, rc, l, lx, "fp32", nbins=nbins, hi=top * rc)
    check(clm, x, H, rc, l, lx, "fp32", nbins=nbins, hi=top * 0.6 * rc, cutoff=0.6 * rc)


def test_clustered_and_coincident(clm):
    """Cells of hundreds of particles beside empty ones, particles at one point,
    pairs of equal velocity."""
    H = np.eye(2)
    g = W.rng(51)
    x = np.concatenate([0.5 + 0.003 * g.normal(size=(1500, 2)), g.random((300, 2)), np.full((70, 2), 0.25)])
    check(clm, x, H, 0.01, 2, None, "fp32")
    cl = clm.CellList(T(x), clm.Box(H, 0.01, 2))
    h, s, c = cl.relspeed_histogram(torch.zeros((len(x), 2), dtype=torch.float64, device="cuda:0"), 8, 2.0)
    n = oracle.compute(x, H, 0.01)["count"]
    assert int(c.item()) == n and h.tolist() == [n] + [0] * 8 and float(s.abs().sum()) == 0.0


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("box", list(BOXES))
@pytest.mark.parametrize("n", [1, 16, 17, 65, 1000, 4001])
def test_force_gather(clm, box, n, precision):
    """The force gather (every pair from both ends): forces per particle against
    the sum of its pair-force magnitudes (1e-5 / 1e-11), energy, box gradient
    and virial against the largest force sum (wrapped and image particles)."""
    H, rc, l, lx = BOXES[box]
    dim = H.shape[0]
    x = W.uniform_in_box(n, H, 700 + n) + H @ (np.arange(dim) % 2 * 2.0 - 1.0)
    x[::3] += H @ np.full(dim, 2.0)   # a third of the particles two boxes away
    sigma, eps = 0.3 * rc, 0.3
    ref = oracle.compute(x, H, rc, lj=(sigma, eps), lj_grad=True, lj_fabs=True)
    cl = clm.CellList(T(x), clm.Box(H, rc, l, lcell_x=lx), precision=precision)
    tol_e, tol_f = (1e-6, 1e-5) if precision == "fp32" else (1e-12, 1e-11)
    for virial in (False, True):
        out = cl.lj_forces(sigma, eps, virial=virial, half=False)
        assert int(out["count"].item()) == ref["count"]
        # sum of |u|: at most |E| and twice the negative terms, each above -eps
        assert abs(out["energy"].item() - ref["lj_energy"]) <= tol_e * (abs(ref["lj_energy"]) + 2 * eps * ref["count"])
        err = np.linalg.norm(out["forces"].cpu().numpy() + ref["lj_grad"], axis=1)
        assert np.all(err <= tol_f * ref["lj_fabs"])
        # f D M^T and f D D^T: at most the force sum times |M| (images and wraps: 4) / the cutoff
        top = ref["lj_fabs"].sum()
        assert np.abs(out["grad_box"].cpu().numpy() - ref["dEdH"]).max() <= tol_f * 4 * top
        if virial:
            assert np.abs(out["virial"].cpu().numpy() - ref["virial"]).max() <= tol_f * rc * top


SPARSE = {"3d": (np.diag([60.0, 60.0, 60.0]), 1.0, 3), "2d": (np.diag([400.0, 380.0]), 1.5, 2)}


def sparse_points(name, seed):
    """Mostly a particle or two a tile (a wave takes a whole tile), and clumps whose tiles are full."""
    H, rc, dim = SPARSE[name]
    x = W.uniform_in_box(12000, H, seed)
    clump = np.full(dim, 20.0) + W.rng(seed + 1).normal(scale=1.5, size=(700, dim))
    return np.concatenate([x, clump]), H, rc


@pytest.mark.parametrize("name", list(SPARSE))
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_sparse_box(clm, name, precision):
    x, H, rc = sparse_points(name, 31)
    check(clm, x, H, rc, 2, None, precision)
    y = W.uniform_in_box(9000, H, 33)
    check(clm, x, H, rc, 2, None, precision, y=y)


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_cells_of_many_particles(clm, dim, precision):
    """Buckets of the build that hold too many particles to be assembled in LDS:
    their cells are ordered along a curve."""
    L, m, s = (100.0, 5000, 2.5) if dim == 2 else (40.0, 6000, 2.0)
    H = np.eye(dim) * L
    x = np.concatenate([W.uniform_in_box(17000, H, 71), (0.4 * L + W.rng(72).normal(scale=s, size=(m, dim))) % L])
    check(clm, x, H, 5.0, 2, None, precision)
