"""Sorted neighbour lists by rows: the same pairs and, bit for bit, the same
distances as the unsorted list, over boxes, sizes, lengths of rows (each side of
what a wave, a block and one window of the longest rows hold) and capacities.
Everything here is exact, so there is no tolerance."""
import ctypes

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


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


BOXES = {
    "tri3": (W.triclinic_h((31.0, 30.0, 33.0), (80.0, 95.0, 100.0)), 5.0, 2, None),
    "fewest3": (np.diag([30.0, 30.0, 30.0]), 11.5, 2, None),   # five cells on an axis
    "row3": (np.diag([200.0, 9.1, 9.1]), 3.0, 1, 4),           # long rows, three cells across
    "cells3": (np.diag([500.0, 9.1, 9.1]), 3.0, 1, 8),         # groups over more than 64 cells
    "tri2": (np.array([[55.0, -12.0], [0.0, 50.0]]), 6.0, 2, None),
    "l1_2": (np.diag([40.0, 40.0]), 13.0, 1, None),            # three cells on an axis
}


def in_order(pairs, dist):
    p, d = pairs.cpu().numpy().astype(np.int64), dist.cpu().numpy()
    o = np.lexsort((p[:, 1], p[:, 0]))
    return p[o], d[o]


def check(cl, ref=None, **kw):
    p, d = cl.neighbor_list(sorted=True, **kw)
    wp, wd = in_order(*cl.neighbor_list(**kw))
    assert np.array_equal(p.cpu().numpy(), wp)
    assert np.array_equal(d.cpu().numpy(), wd)
    p, _ = cl.neighbor_list(sorted=True, distances=False, **kw)
    assert np.array_equal(p.cpu().numpy(), wp)
    if ref is not None:
        assert np.array_equal(wp[:, 0], ref["nl_i"]) and np.array_equal(wp[:, 1], ref["nl_j"])


@pytest.mark.parametrize("box", list(BOXES))
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_rows_match_the_unsorted_list(clm, box, precision):
    H, rc, l, lx = BOXES[box]
    for n in (6, 17, 65, 1500):
        print(f"case {box} {precision} n={n}", flush=True)
        x = W.uniform_in_box(n, H, 40 + n) + H @ np.full(H.shape[0], 2.0)
        y = W.uniform_in_box(3 * n + 1, H, 41 + n)
        b = clm.Box(H, rc, l, lcell_x=lx)
        check(clm.CellList(T(x), b, precision=precision), oracle.compute(x, H, rc, nl=True))
        check(clm.CellList(T(x), b, y=T(y), precision=precision), oracle.compute(x, H, rc, y, nl=True))
        check(clm.CellList(T(x), b, precision=precision), oracle.compute(x, H, 0.7 * rc, nl=True), cutoff=0.7 * rc)


@pytest.mark.parametrize("lengths", [(1, 2, 63, 64, 65, 128), (511, 512, 513, 1023, 1024, 1025, 2049), (8191, 8192, 8193),
                                     (270000, 3)])
def test_lengths_of_rows(clm, lengths):
    H, rc = np.diag([120.0, 40.0, 40.0]), 6.0
    r = W.rng(5)
    c = np.array([[10.0 + 14.0 * k, 11.0, 12.0] for k in range(8)])
    y = np.concatenate([c[k] + r.uniform(-1.7, 1.7, size=(m, 3)) for k, m in enumerate(lengths)])
    who = np.repeat(np.arange(len(lengths)), lengths)
    o = r.permutation(len(y))
    cl = clm.CellList(T(c), clm.Box(H, rc, 2), y=T(y[o]), precision="fp32")
    p, d = cl.neighbor_list(sorted=True)
    p, d = p.cpu().numpy(), d.cpu().numpy()
    want = np.lexsort((np.arange(len(o)), who[o]))
    assert np.array_equal(p[:, 0], who[o][want]) and np.array_equal(p[:, 1], want)
    wp, wd = in_order(*cl.neighbor_list())
    assert np.array_equal(p, wp) and np.array_equal(d, wd)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_list_beyond_its_capacity(clm, precision):
    L = clm._lib
    H, rc, l, lx = BOXES["tri3"]
    x = W.uniform_in_box(3000, H, 8)
    cl = clm.CellList(T(x), clm.Box(H, rc, l), precision=precision)
    p, d = cl.neighbor_list(sorted=True)
    p, d = p.cpu().numpy(), d.cpu().numpy()
    for cap in (1, 1000, len(p) - 1):
        need = ctypes.c_size_t(0)
        L.check(L.lib().clm_pairs_sort_workspace_bytes(cap, 1, ctypes.byref(need)))
        ws = torch.empty(int(need.value) + 256, dtype=torch.uint8, device="cuda:0")
        pairs = torch.full((cap + 64, 2), -7, dtype=torch.int32, device="cuda:0")
        dist = torch.full((cap + 64,), -7.0, dtype=torch.float64, device="cuda:0")
        c = torch.full((1,), -1, dtype=torch.int64, device="cuda:0")
        ptr = lambda t: ctypes.c_void_p(t.data_ptr())
        P = L.MapParams(capacity=cap, with_distances=1, sorted=1, scratch_bytes=int(need.value),
                        scratch_dev=ctypes.c_void_p(ws.data_ptr() + (-ws.data_ptr()) % 256))
        O = L.MapOut(pairs_dev=ptr(pairs), dist_dev=ptr(dist), count_dev=ptr(c))
        L.check(L.lib().clm_map(cl._h, L.MAP_KINDS["neighbor_list"], ctypes.byref(P), ctypes.byref(O)))
        torch.cuda.synchronize()
        assert int(c.item()) == len(p)
        gp, gd = pairs.cpu().numpy(), dist.cpu().numpy()
        assert (gp[cap:] == -7).all() and (gd[cap:] == -7.0).all()
        whole = np.searchsorted(p[:, 0], p[cap, 0])  # the rows before the one that is cut
        assert np.array_equal(gp[:whole], p[:whole]) and np.array_equal(gd[:whole], d[:whole])
        # of the cut row, entries of the list in ascending order
        row = {tuple(a): b for a, b in zip(p, d)}
        cut = [tuple(a) for a in gp[whole:cap]]
        assert cut == sorted(set(cut)) and all(row[a] == b for a, b in zip(cut, gd[whole:cap]))


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_sparse_box(clm, precision):
    H, rc = np.diag([60.0, 60.0, 60.0]), 1.0
    x = np.concatenate([W.uniform_in_box(12000, H, 31), 20.0 + W.rng(32).normal(scale=1.5, size=(700, 3))])
    b = clm.Box(H, rc, 2)
    check(clm.CellList(T(x), b, precision=precision), oracle.compute(x, H, rc, nl=True))
    y = W.uniform_in_box(9000, H, 33)
    check(clm.CellList(T(x), b, y=T(y), precision=precision), oracle.compute(x, H, rc, y, nl=True))
