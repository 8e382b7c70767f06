"""Batches of so many graphs that a level's tables (38 bytes a graph) do not fit the
context's pinned staging buffer of 256 KiB, and on either side of that, against the
oracle graph by graph."""
import numpy as np
import pytest

import oracle
from paper_2204_02934_amd import graphs

pytestmark = pytest.mark.gpu


def _kinds():
    """Eleven small graphs that coarsen once, twice or not at all, and what they give."""
    gs = [graphs.edgeless(1), graphs.path(2), graphs.path(9), graphs.cycle(30), graphs.star(12),
          graphs.complete(7), graphs.grid2d_5pt(6, 5), graphs.edgeless(5), graphs.path(41),
          graphs.grid2d_5pt(9, 3), graphs.grid3d_7pt(3, 3, 4)]
    return gs, [oracle.coarsen(rp, c, seed=2, stop_below=4) for rp, c in gs]


@pytest.mark.parametrize("n_graphs", [6889, 6890, 9000])  # the first that fits, the first that does not
def test_batch(n_graphs):
    from paper_2204_02934_amd import api
    gs, want = _kinds()
    pick = np.random.default_rng(n_graphs).integers(0, len(gs), n_graphs)
    counts = np.concatenate([np.diff(gs[k][0]) for k in pick])
    voff = np.concatenate([[0], np.cumsum([gs[k][0].size - 1 for k in pick])])
    rp = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    col = np.concatenate([gs[k][1] + voff[i] for i, k in enumerate(pick)]).astype(np.int32)
    got = api.Context(0).aggregate_batched(rp, col, voff, seed=2, stop_below=4)
    assert len(got) == n_graphs
    for k, levels in zip(pick, got):
        assert [(l["n"], l["nnz"], l["n_agg"]) for l in levels] == \
            [(l["n"], l["nnz"], l["n_agg"]) for l in want[k]]
        for a, b in zip(levels, want[k]):
            assert np.array_equal(a["agg"].cpu().numpy(), b["agg"])
