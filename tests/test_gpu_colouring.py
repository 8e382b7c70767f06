"""GPU parity of the colouring and the sweep order behind mis2_cgs_setup at the
limits of their kernels: 64 colours and one more (the counting sort's limit), a
second window of 64 colours, tiles of 2048 ids and wavefronts of one vertex
more or less, clusters of 64 / 65 and 512 / 513 rows, lists that outlive many launches."""
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


CASES = {
    "k64": lambda: graphs.complete(64),
    "k65": lambda: graphs.complete(65),
    "k130": lambda: graphs.complete(130),  # a dependence chain of every vertex
    "one": lambda: graphs.edgeless(1),
    "path2047": lambda: graphs.path(2047),
    "path2048": lambda: graphs.path(2048),
    "path2049": lambda: graphs.path(2049),
    "grid8193": lambda: graphs.grid2d_5pt(8193, 1),
    "grid27": lambda: graphs.grid3d_27pt(31, 29, 33),
    "elasticity": lambda: graphs.elasticity3d(9, 10, 11),
    "star64": lambda: graphs.disjoint_union([graphs.star(64), graphs.star(65), graphs.star(66)]),
    "star511": lambda: graphs.disjoint_union([graphs.star(511), graphs.star(512), graphs.star(513)]),
    "chunglu": lambda: graphs.chung_lu(70_000, 12.0, 2.1, 3000, seed=8),
}


@pytest.mark.parametrize("point", [False, True])
@pytest.mark.parametrize("name", sorted(CASES))
def test_plan(ctx, name, point):
    rp, c = CASES[name]()
    n = rp.size - 1
    want = oracle.cgs_plan(rp, c, 5, point=point)
    plan = ctx.cgs_setup(rp, c, seed=5, point=point)
    k = want["n_clusters"]
    assert (plan.n_clusters, plan.n_colors) == (k, want["n_colors"])
    for got, key in ((plan.cluster[:n], "cluster"), (plan.cluster_color[:k], "cluster_color"),
                     (plan.rows[:n], "rows"), (plan.cluster_off[:k + 1], "cluster_off")):
        assert np.array_equal(got.cpu().numpy(), want[key]), key
    inv = np.empty(n, np.int32)
    inv[want["rows"]] = np.arange(n, dtype=np.int32)
    assert np.array_equal(plan.pos.cpu().numpy()[:n], inv)
    assert np.array_equal(plan.color_off[:plan.n_colors + 1], want["color_off"])
