"""Round 0's Decide Set with staged rows on either side of the rule that gives it
the list of rows to read (2^17 vertices, or 16 entries a vertex), in one or many
segments, against the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_2204_02934_amd import graphs

pytestmark = pytest.mark.gpu

N = 1 << 17


def _ring(n, k):
    """Every vertex joined to the k next ones on a ring: 2 k entries a vertex."""
    u = np.repeat(np.arange(n), k)
    return graphs.from_edges(n, u, (u + np.tile(np.arange(1, k + 1), n)) % n)


GRAPHS = {
    "below": lambda: graphs.disjoint_union([graphs.path(N // 2 - 1), graphs.edgeless(N // 2)]),
    "at": lambda: graphs.disjoint_union([graphs.path(N // 2), graphs.edgeless(N // 2)]),
    "entries14": lambda: _ring(9001, 7),
    "entries16": lambda: _ring(9001, 8),
}


@pytest.mark.parametrize("blocks", [1, 0])
@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_aggregate(name, blocks):
    from paper_2204_02934_amd import api
    rp, c = GRAPHS[name]()
    want, n_agg = oracle.aggregate(rp, c, 2)
    agg, na = api.Context(0, lanes=-2, blocks=blocks).aggregate(rp, c, 2)
    assert na == n_agg and np.array_equal(agg.cpu().numpy(), want)
