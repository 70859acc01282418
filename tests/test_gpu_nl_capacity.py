"""A sorted list longer than its capacity holds the first `capacity` pairs of the
whole list, the same ones on every call, and the count is the whole list's:
capacities at and around the ends of rows, within rows of every length class
(a wave's, a block's, longer), one and two sets.  Exact."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def clm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2202_06427_amd as clm
    return clm


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def partial(clm, cl, cap, distances):
    L = clm._lib
    need = ctypes.c_size_t(0)
    L.check(L.lib().clm_pairs_sort_workspace_bytes(cap, distances, ctypes.byref(need)))
    ws = torch.empty(int(need.value) + 256, dtype=torch.uint8, device="cuda:0")
    pairs = torch.full((cap + 64, 2), -7, dtype=torch.int32, device="cuda:0")
    dist = torch.full((cap + 64,), -7.0, dtype=torch.float64, device="cuda:0")
    c = torch.full((1,), -1, dtype=torch.int64, device="cuda:0")
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    P = L.MapParams(capacity=cap, with_distances=distances, sorted=1, scratch_bytes=int(need.value),
                    scratch_dev=ctypes.c_void_p(ws.data_ptr() + (-ws.data_ptr()) % 256))
    O = L.MapOut(pairs_dev=ptr(pairs), dist_dev=ptr(dist), count_dev=ptr(c))
    L.check(L.lib().clm_map(cl._h, L.MAP_KINDS["neighbor_list"], ctypes.byref(P), ctypes.byref(O)))
    torch.cuda.synchronize()
    return pairs.cpu().numpy(), dist.cpu().numpy(), int(c.item())


def check(clm, cl, caps):
    p, d = (t.cpu().numpy() for t in cl.neighbor_list(sorted=True))
    for cap in caps(p[:, 0]):
        if not 0 < cap < len(p):
            continue
        for distances in (1, 0, 1):
            gp, gd, c = partial(clm, cl, cap, distances)
            assert c == len(p)
            assert np.array_equal(gp[:cap], p[:cap]) and (gp[cap:] == -7).all(), cap
            if distances:
                assert np.array_equal(gd[:cap], d[:cap]) and (gd[cap:] == -7.0).all(), cap


def around_rows(i):
    ends = np.flatnonzero(np.diff(i)) + 1
    pick = ends[:: max(1, len(ends) // 5)]
    return [1, 2, len(i) // 3, len(i) - 1] + [int(e) + k for e in pick for k in (-1, 0, 1)]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_one_set(clm, precision):
    H = W.triclinic_h((31.0, 30.0, 33.0), (80.0, 95.0, 100.0))
    for n in (8, 9, 40, 3000):
        x = W.uniform_in_box(n, H, 8)
        check(clm, clm.CellList(T(x), clm.Box(H, 5.0, 2), precision=precision), around_rows)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_two_sets(clm, precision):
    H = W.triclinic_h((31.0, 30.0, 33.0), (80.0, 95.0, 100.0))
    for n, m in ((1, 3000), (300, 5), (400, 4001)):
        cl = clm.CellList(T(W.uniform_in_box(n, H, 8)), clm.Box(H, 5.0, 2), y=T(W.uniform_in_box(m, H, 9)),
                          precision=precision)
        check(clm, cl, around_rows)


def test_lengths_of_the_cut_row(clm):
    H, r = np.diag([120.0, 40.0, 40.0]), W.rng(5)
    lengths = (3, 700, 1100, 9000, 270000, 40)
    c = np.array([[10.0 + 14.0 * k, 11.0, 12.0] for k in range(len(lengths))])
    y = np.concatenate([c[k] + r.uniform(-1.7, 1.7, size=(m, 3)) for k, m in enumerate(lengths)])
    cl = clm.CellList(T(c), clm.Box(H, 6.0, 2), y=T(y[r.permutation(len(y))]), precision="fp32")
    starts = np.cumsum((0,) + lengths)
    check(clm, cl, lambda i: [int(s + f * m) for s, m in zip(starts, lengths) for f in (0.3, 0.999)])


def test_dense_rows_of_a_sparse_box(clm):
    H = np.diag([60.0, 60.0, 60.0])
    x = np.concatenate([W.uniform_in_box(12000, H, 31), 20.0 + W.rng(32).normal(scale=1.5, size=(700, 3))])
    check(clm, clm.CellList(T(x), clm.Box(H, 1.0, 2), precision="fp32"), around_rows)
