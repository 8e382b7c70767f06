"""GPU quotient graphs of labellings with vertices that belong to no aggregate
(label -1, dropped) and aggregates without a vertex, against a plain set of the
couplings.  The workspace is filled with large words first, so an index read
from memory that nothing wrote would leave every array."""
import numpy as np
import pytest

from paper_2204_02934_amd import graphs

pytestmark = pytest.mark.gpu


def _couplings(rp, c, agg, n_agg):
    row = np.repeat(agg, np.diff(rp))
    other = agg[c]
    keep = (row >= 0) & (other >= 0) & (row != other)
    key = np.unique(row[keep].astype(np.int64) * max(n_agg, 1) + other[keep])
    crow = np.zeros(n_agg + 1, np.int64)
    np.cumsum(np.bincount(key // max(n_agg, 1), minlength=n_agg), out=crow[1:])
    return crow, (key % max(n_agg, 1)).astype(np.int32)


def _labels(name, n):
    agg = np.full(n, -1, np.int32)
    rng = np.random.default_rng(3)
    if name == "first":  # one vertex in the first of n aggregates
        agg[n // 2] = 0
        return agg, n
    if name == "last":
        agg[0] = n - 1
        return agg, n
    if name == "some":  # two of three vertices, every second aggregate empty
        pick = rng.random(n) < 0.67
        agg[pick] = 2 * rng.integers(0, n // 8, pick.sum())
        return agg, n // 4
    return agg, {"none1": 1, "none": n // 3, "none_n": n}[name]


# 16 lanes a row or 64 (more than 256 entries an aggregate), and past the member
# kernel of small graphs
GRAPHS = {
    "grid": lambda: graphs.grid2d_5pt(40, 30),
    "dense": lambda: graphs.complete(300),
    "large": lambda: graphs.grid3d_7pt(25, 26, 27),
}


@pytest.mark.parametrize("labels", ["none1", "none", "none_n", "first", "last", "some"])
@pytest.mark.parametrize("graph", sorted(GRAPHS))
def test_quotient(graph, labels):
    from paper_2204_02934_amd import _lib, api
    rp, c = GRAPHS[graph]()
    agg, n_agg = _labels(labels, rp.size - 1)
    ctx = api.Context(0)
    ctx.ensure_workspace(rp.size - 1, _lib.MIS2_OP_COARSEN).fill_(0x7F)
    crow, ccol = ctx.quotient(rp, c, agg, n_agg)
    want_row, want_col = _couplings(rp, c, agg, n_agg)
    assert np.array_equal(crow.cpu().numpy(), want_row)
    assert np.array_equal(ccol.cpu().numpy(), want_col)
