"""The scan of the tile counts (2048 vertices a tile) at the numbers of tiles where
it takes one, two, four or eight rows of 256: the MIS-2 count, and a point plan of
more than 64 colours, whose rows are listed colour by colour through it."""
import numpy as np
import pytest

from paper_2204_02934_amd import graphs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [1, 255, 256, 257, 512, 513, 1024, 1025, 2048, 2049])
def test_count_and_order(tiles):
    from paper_2204_02934_amd import api
    n = 2048 * (tiles - 1) + 700  # the last tile in part
    k = 66
    u, v = np.triu_indices(k, 1)  # 66 colours
    w = np.arange(k, n - 1, 3)    # and pairs with a vertex alone between them
    rp, c = graphs.from_edges(n, np.concatenate([u, w]), np.concatenate([v, w + 1]))
    print("n", n, "entries", c.size, flush=True)
    ctx = api.Context(0)
    status, n_roots, _ = ctx.mis2(rp, c, 1)
    assert n_roots == int(status.sum().item()) == 1 + w.size + (n - k - 2 * w.size)
    plan = ctx.cgs_setup(rp, c, 1, point=True)
    color = plan.cluster_color.cpu().numpy()
    assert color.max() >= 65
    assert np.array_equal(plan.rows.cpu().numpy(), np.argsort(color, kind="stable"))
