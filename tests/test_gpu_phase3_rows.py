"""GPU parity of phase 3 where a row couples to many aggregates: as many as a
wavefront counts one by one and one more, every neighbour in another aggregate,
ties decided by size and by id, rows of 128 and 129 entries, and the sizes of the
workgroup's map, against the oracle's labels."""
import numpy as np
import pytest

import oracle
from paper_2204_02934_amd import graphs
from test_gpu_phase3 import _late, _split

pytestmark = pytest.mark.gpu


def _shares(total, parts):
    """A row of `total` neighbours over `parts` aggregates, the rest in the last."""
    return [total // parts] * (parts - 1) + [total - total // parts * (parts - 1)]


CASES = {
    # 7, 8, 9 and 10 aggregates, the last one the best or none better than another
    "few": lambda: _late([_shares(t, p) for t in (33, 64, 65, 128) for p in (7, 8, 9, 10)]),
    "distinct": lambda: _late([[1] * t for t in (33, 63, 64, 65, 127, 128, 129)]),
    "ties": lambda: _late([[2] * 9 + [1] * 20, [1] * 60 + [2] * 2, [3] * 30, [4] * 16 + [1] * 64,
                           [1] * 126 + [2]]),
    "map": lambda: _late([_split(t, 3, t) for t in
                          (129, 255, 256, 257, 511, 512, 513, 1024, 1025, 2048, 2049, 4095)]),
    "map_distinct": lambda: _late([[1] * 257 + [2], [1] * 512, [1] * 1025 + [2] * 2, [1] * 4095]),
    # nothing for the workgroup: no row of more than 128 entries
    "to_128": lambda: _late([_split(t, 4, t) for t in range(30, 129, 7)] + [[1] * 128]),
    "elasticity": lambda: graphs.elasticity3d(13, 15, 14),
}


@pytest.mark.parametrize("lanes", [0, 1, 2, 4, 8, 64, -1, -2])
@pytest.mark.parametrize("name", sorted(CASES))
def test_aggregate(name, lanes):
    from paper_2204_02934_amd import api
    rp, c = CASES[name]()
    want, n_agg = oracle.aggregate(rp, c, 0)
    for autotune in (True, False):  # (small graphs: one workgroup, or launched)
        got, na = api.Context(0, lanes=lanes, autotune=autotune).aggregate(rp, c, 0)
        assert na == n_agg
        assert np.array_equal(got.cpu().numpy(), want)


def test_persistent():
    from paper_2204_02934_amd import api
    rp, c = CASES["map"]()
    want, n_agg = oracle.aggregate(rp, c, 0)
    got, na = api.Context(0, persistent=True).aggregate(rp, c, 0)
    assert na == n_agg and np.array_equal(got.cpu().numpy(), want)
