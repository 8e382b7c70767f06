"""Round 0's Decide Set with a list of the rows that have to be read: segments with
none, some and more of them than the list holds, masked and unmasked, at every
lane count that takes it.  Status, rounds and aggregates must equal the CPU
oracle's."""
import numpy as np
import pytest

import oracle
from paper_2204_02934_amd import graphs

pytestmark = pytest.mark.gpu

GRAPHS = {
    # every vertex is its own neighbourhood's least: all rows are read
    "edgeless": lambda: graphs.edgeless(300_000),
    # most are
    "pairs": lambda: graphs.from_edges(200_000, np.arange(0, 200_000, 8), np.arange(1, 200_000, 8)),
    "grid27": lambda: graphs.grid3d_27pt(30, 29, 28),
    "chunglu": lambda: graphs.chung_lu(30_000, 20.0, 2.1, 3000, seed=4),
    "mixed": lambda: graphs.disjoint_union([graphs.edgeless(40_000), graphs.grid3d_7pt(20, 20, 20),
                                            graphs.edgeless(3000), graphs.complete(300),
                                            graphs.star(9000, 17)]),
}


@pytest.mark.parametrize("blocks", [8, 0])  # long segments, and as many as usual
@pytest.mark.parametrize("lanes", [-2, -1, 4, 8, 16, 64])
@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_rows_to_read(name, lanes, blocks):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2204_02934_amd import _lib, api
    print(name, "lanes", lanes, "blocks", blocks, flush=True)
    rp, c = GRAPHS[name]()
    ctx = api.Context(0, lanes=lanes)
    if blocks:
        ctx.set_option(_lib.MIS2_OPT_GRID_BLOCKS, blocks)
    o = oracle.mis2_ex(rp, c, 5)
    status, _, iters = ctx.mis2(rp, c, 5)
    assert iters == o["n_iters"] and np.array_equal(status.cpu().numpy(), o["status"])
    assert np.array_equal(ctx.last_trace(0), o["trace"][:, :2])
    want, n_want = oracle.aggregate(rp, c, 5)
    agg, n_agg = ctx.aggregate(rp, c, 5)
    assert n_agg == n_want and np.array_equal(agg.cpu().numpy(), want)
