"""The cluster sweep at the edges of its batches (mis2_cgs_apply): rows of every
length class and around the slots of a batch, clusters of several batches, with
the lanes that stage a cluster 16, 64 or 256.  x must equal the CPU oracle's
sequential sweep bit for bit."""
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


def _check(ctx, rp, cc, what, sweeps=2):
    import torch
    n = rp.size - 1
    want = oracle.cgs_plan(rp, cc, 3)
    print(what, "rows", n, "entries per cluster", int(rp[-1]) // want["n_clusters"],
          "largest colour", int(np.diff(want["color_off"]).max()), flush=True)
    plan = ctx.cgs_setup(rp, cc, seed=3)
    val, diag = graphs.matrix_values(rp, cc, 5)
    rng = np.random.default_rng(6)
    b, x0 = rng.standard_normal(n), rng.standard_normal(n)
    dev = torch.device("cuda", 0)
    dval, ddiag, db = (torch.as_tensor(v, device=dev) for v in (val, diag, b))
    for symmetric in (False, True):
        x = torch.as_tensor(x0.copy(), device=dev)
        ctx.cgs_apply(rp, cc, dval, ddiag, plan, db, x, sweeps=sweeps, symmetric=symmetric)
        ref = oracle.cgs_apply(rp, cc, val, diag, want, b, x0, sweeps=sweeps, symmetric=symmetric)
        assert np.array_equal(x.cpu().numpy(), ref), (what, symmetric)
    return int(rp[-1]) // want["n_clusters"], int(np.diff(want["color_off"]).max())


# complete graphs: every row of the one cluster has L entries
@pytest.mark.parametrize("L", [1, 7, 8, 9, 10])
def test_sixteen_lanes(ctx, L):
    per, _ = _check(ctx, *graphs.complete(L + 1), "complete %d" % (L + 1))
    assert per <= 128


@pytest.mark.parametrize("spokes", [127, 128, 129, 300])
def test_sixteen_lanes_long_rows(ctx, spokes):
    # a star among short paths: the hub's row ends at, or is past, the 128 slots
    g = graphs.disjoint_union([graphs.path(5)] * 30 + [graphs.star(spokes + 1, 0)]
                              + [graphs.grid2d_5pt(9, 8)])
    per, _ = _check(ctx, *g, "star %d" % spokes)
    assert per <= 128


@pytest.mark.parametrize("L", [15, 16, 17, 28, 29, 31, 40])
def test_sixty_four_lanes(ctx, L):
    g = graphs.disjoint_union([graphs.complete(L + 1)] * 1030)
    per, wide = _check(ctx, *g, "1030 x complete %d" % (L + 1), sweeps=1)
    assert 128 < per and wide > 1024 and (per <= 1024 or L > 31)


def test_sixty_four_lanes_long_rows(ctx):
    # hubs of 927 .. 929 and 2500 spokes among 1100 cliques
    g = graphs.disjoint_union([graphs.star(k + 1, 0) for k in (927, 928, 929, 2500)]
                              + [graphs.complete(13)] * 1100)
    per, wide = _check(ctx, *g, "stars and cliques", sweeps=1)
    assert 128 < per <= 1024 and wide > 1024


@pytest.mark.parametrize("L", [12, 16, 17, 24, 28, 29, 32, 33, 48, 49, 63, 64, 65, 80, 81, 100])
def test_two_hundred_fifty_six_lanes(ctx, L):
    g = graphs.disjoint_union([graphs.complete(L + 1), graphs.complete(L), graphs.complete(14)])
    per, wide = _check(ctx, *g, "complete %d" % (L + 1))
    assert per > 128 and wide <= 1024


@pytest.mark.parametrize("spokes", [2047, 2048, 2049, 5000])
def test_two_hundred_fifty_six_lanes_long_rows(ctx, spokes):
    per, _ = _check(ctx, *graphs.star(spokes + 1, 0), "star %d" % spokes)
    assert per > 1024
