"""The Galerkin operator at the edges of its two ways of adding: columns one and
two to a lane and past both, items of one and several batches, with a large
aggregate beside them so that the first way is taken, and without.  Everything
must equal the CPU oracle's bit for bit."""
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


def _check(ctx, rp, cc, agg, n_agg, what):
    import torch
    dev = torch.device("cuda", 0)
    print(what, "entries per aggregate", cc.size // n_agg, flush=True)
    val, diag = graphs.matrix_values(rp, cc, 7)
    crp, ccol = oracle.quotient(rp, cc, agg, n_agg)
    _, _, want_val, want_diag = oracle.galerkin(rp, cc, val, diag, agg, n_agg, crp, ccol)
    got_val, got_diag = ctx.galerkin(rp, cc, torch.as_tensor(val, device=dev),
                                     torch.as_tensor(diag, device=dev), agg, crp, ccol)
    assert np.array_equal(got_diag.cpu().numpy(), want_diag), what
    assert np.array_equal(got_val.cpu().numpy()[:want_val.size], want_val), what
    return cc.size // n_agg


def _beside(g, agg, clique):
    """The graph beside one complete graph that is an aggregate of its own."""
    if not clique:
        return (*g, agg, int(agg.max()) + 1)
    rp, cc = graphs.disjoint_union([g, graphs.complete(clique)])
    na = int(agg.max()) + 1
    return rp, cc, np.concatenate([agg, np.full(clique, na)]).astype(np.int32), na + 1


@pytest.mark.parametrize("clique", [0, 250])
@pytest.mark.parametrize("columns", [1, 2, 3, 63, 64, 65, 125, 126, 127, 255, 256])
def test_columns(ctx, columns, clique):
    # a hub and a friend, joined, and one aggregate for each of the hub's leaves
    n = columns + 2
    u = np.concatenate([np.zeros(columns + 1, np.int64), np.ones(columns // 2, np.int64)])
    v = np.concatenate([1 + np.arange(columns + 1), 2 + np.arange(columns // 2)])
    g = graphs.from_edges(n, u, v)
    agg = np.concatenate([[0, 0], 1 + np.arange(columns)]).astype(np.int32)
    per = _check(ctx, *_beside(g, agg, clique), "columns %d" % columns)
    assert (per > 200) == (clique > 0)


@pytest.mark.parametrize("clique", [0, 60])
@pytest.mark.parametrize("leaves", [1, 15, 16, 17, 63, 64, 65, 126, 127, 128, 255, 256, 257, 1000])
def test_items(ctx, leaves, clique):
    # the hub's one column takes `leaves` items, the leaves' one of each of theirs
    g = graphs.star(leaves + 1, 0)
    agg = np.ones(leaves + 1, np.int32)
    agg[0] = 0
    _check(ctx, *_beside(g, agg, clique), "leaves %d" % leaves)


@pytest.mark.parametrize("parts", [1, 2, 5, 90, 130])
def test_random_columns(ctx, parts):
    # every aggregate meets every other many times, in no order
    rp, cc = graphs.random_regular_ish(2000, 40, seed=parts)
    agg = (np.random.default_rng(parts).permutation(2000) % parts).astype(np.int32)
    assert _check(ctx, rp, cc, agg, parts, "parts %d" % parts) > 200
