"""Aggregation of graphs whose roots are numbered through the scan of the tile
counts (more than 4096 tiles of 2048 vertices; 2048 tiles a step).  Vertex counts
at steps' ends and one past; labels must equal the CPU oracle's."""
import numpy as np
import pytest

import oracle
from paper_2204_02934_amd import graphs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles,extra", [(2 * 2048, 0), (2 * 2048, 1), (3 * 2048, 0)])
def test_roots_past_a_step(tiles, extra):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2204_02934_amd import api
    n = 2048 * tiles + extra
    rng = np.random.default_rng(tiles + extra)
    u = rng.integers(0, n, n // 8)
    v = np.minimum(u + rng.integers(1, 50, u.size), n - 1)
    keep = u != v
    rp, c = graphs.from_edges(n, u[keep], v[keep])
    print("n", n, "entries", c.size, flush=True)
    want, want_n = oracle.aggregate(rp, c, 5)
    agg, n_agg = api.Context(0).aggregate(rp, c, 5)
    assert n_agg == want_n and np.array_equal(agg.cpu().numpy(), want)
