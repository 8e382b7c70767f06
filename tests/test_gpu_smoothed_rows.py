"""Smoothed aggregation at the edges of its row classes (mis2_smoothed): rows of
P sorted in registers or collected in a set, rows of A P and of the coarse
operator in each of the three sets, P written with and without room for a spare
copy, and columns of P longer than each of the member sorts takes.  Everything
must equal the CPU oracle's bit for bit."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2204_02934_amd import graphs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2204_02934_amd import api
    return api.Context(0)


def _spokes(s):
    """A hub with s spokes of three vertices each, every spoke its own aggregate
    and the hub another: s + 1 columns in the hub's row of P, of A P and of the
    coarse operator, s entries in its row of A."""
    a = 1 + 3 * np.arange(s)
    rp, c = graphs.from_edges(1 + 3 * s, np.concatenate([np.zeros(s, np.int64), a, a + 1]),
                              np.concatenate([a, a + 1, a + 2]))
    return rp, c, np.concatenate([[0], 1 + np.repeat(np.arange(s), 3)]).astype(np.int32), s + 1


def _dense_spokes(s):
    """The same beside complete graphs, with more than seven entries a row."""
    rp, c, agg, na = _spokes(s)
    k = 5
    rp2, c2 = graphs.disjoint_union([(rp, c)] + [graphs.complete(20)] * k)
    assert c2.size > 7 * (rp2.size - 1)
    return rp2, c2, np.concatenate([agg, na + np.repeat(np.arange(k), 20)]).astype(np.int32), na + k


def _call(ctx, rp, c, val, diag, agg, na, omega):
    import torch
    dev = torch.device("cuda", 0)
    (a, b, d), (e, f, g) = ctx.smoothed(rp, c, torch.as_tensor(val, device=dev),
                                        torch.as_tensor(diag, device=dev), agg, na, omega)
    return [x.cpu().numpy() for x in (a, b, d, e, f, g)]


def _check(ctx, rp, c, agg, na, seed):
    val, diag = graphs.matrix_values(rp, c, seed, shift=0.25)
    want = oracle.smoothed(rp, c, val, diag, agg, na, 2.0 / 3.0)
    got = _call(ctx, rp, c, val, diag, agg, na, 2.0 / 3.0)
    for k, (g, w) in enumerate(zip(got, want)):
        assert g.shape == w.shape and np.array_equal(g, w), k
    return want


@pytest.mark.parametrize("s", [6, 7, 8, 15, 16, 46, 47, 94, 95, 158, 159, 511, 512, 2047])
def test_row_classes(ctx, s):
    print("spokes", s, flush=True)
    rp, c, agg, na = _spokes(s)
    want = _check(ctx, rp, c, agg, na, s)
    assert want[0][1] == s + 1 and want[3][1] == s + 1


@pytest.mark.parametrize("s", [7, 8, 14, 15, 16])
def test_row_classes_among_dense_rows(ctx, s):
    print("dense spokes", s, flush=True)
    _check(ctx, *_dense_spokes(s), s)


def test_row_past_the_limit(ctx):
    from paper_2204_02934_amd._lib import Mis2Error
    rp, c, agg, na = _spokes(2048)
    val, diag = graphs.matrix_values(rp, c, 1, shift=0.25)
    with pytest.raises(Mis2Error, match="2048 columns"):
        _call(ctx, rp, c, val, diag, agg, na, 0.5)


@pytest.mark.parametrize("m", [128, 129, 512, 513, 4096, 4097])
def test_long_columns(ctx, m):
    # the hub is an aggregate, its m - 1 spokes the other: two columns of m entries
    print("column", m, flush=True)
    rp, c = graphs.from_edges(m, np.zeros(m - 1, np.int64), 1 + np.arange(m - 1))
    agg = np.ones(m, np.int32)
    agg[0] = 0
    want = _check(ctx, rp, c, agg, 2, m)
    assert np.array_equal(np.bincount(want[1]), [m, m])


@pytest.mark.parametrize("graph", ["7pt", "27pt", "spokes"])
@pytest.mark.parametrize("room", ["exact", "half", "half+1"])
def test_room_for_p(ctx, graph, room):
    """P's structure is written once where its value array has room for
    (n + nnz) / 2 values, in a second pass where it has not."""
    import torch
    if graph == "spokes":
        rp, c, agg, na = _spokes(600)
    else:
        make = graphs.grid3d_7pt if graph == "7pt" else graphs.grid3d_27pt
        rp, c = make(11, 10, 9)
        agg, na = oracle.aggregate(rp, c, 0)
    n, nnz = rp.size - 1, c.size
    val, diag = graphs.matrix_values(rp, c, 3, shift=0.25)
    want = oracle.smoothed(rp, c, val, diag, agg, na, 0.5)
    pn, cn = want[1].size, want[4].size
    p_cap = {"exact": pn, "half": max(pn, (n + nnz) // 2 - 3),
             "half+1": max(pn, (n + nnz) // 2 + 4)}[room]
    print(graph, room, p_cap, (n + nnz) // 2, flush=True)
    dev = torch.device("cuda", 0)
    g, keep = ctx.graph(rp, c)
    dval, ddiag = torch.as_tensor(val, device=dev), torch.as_tensor(diag, device=dev)
    dagg = torch.as_tensor(np.asarray(agg, np.int32), device=dev)
    out = [torch.zeros(k + 8, dtype=t, device=dev)
           for k, t in ((n + 1, torch.int64), (p_cap, torch.int32), (p_cap, torch.float64),
                        (na + 1, torch.int64), (cn, torch.int32), (cn, torch.float64))]
    for x in out:
        x[-8:] = -77  # a guard past each array
    ptr = [ctypes.c_void_p(x.data_ptr()) for x in out]
    got_p, got_c, need = ctypes.c_int64(0), ctypes.c_int64(0), ctypes.c_size_t(0)
    for _ in range(6):
        need.value = 0
        rc = ctx.lib.mis2_smoothed(
            ctx.ptr, ctypes.byref(g), ctypes.c_void_p(dval.data_ptr()),
            ctypes.c_void_p(ddiag.data_ptr()), ctypes.c_void_p(dagg.data_ptr()), int(na),
            ctypes.c_double(0.5), ptr[0], ptr[1], ptr[2], p_cap, ptr[3], ptr[4], ptr[5], cn,
            ctypes.byref(got_p), ctypes.byref(got_c), ctypes.byref(need), None)
        if not need.value:
            break
        ctx._ensure_bytes(need.value)
    assert rc == 0 and (got_p.value, got_c.value) == (pn, cn)
    torch.cuda.synchronize()
    sizes = (n + 1, pn, pn, na + 1, cn, cn)
    for k, (x, w, m) in enumerate(zip(out, want, sizes)):
        assert np.array_equal(x[:m].cpu().numpy(), w), k
        assert (x[-8:] == -77).all(), k
    del keep
