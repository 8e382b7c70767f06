"""Rounds whose tuples are computed, one lane per row, on rows of very different
lengths: around the lanes' batch of 8, the cooperative threshold of 32 and the
4096 entries past which the wavefront takes a row, single and side by side.
Status and aggregates must equal the CPU oracle's."""
import numpy as np
import pytest

import oracle
from paper_2204_02934_amd import graphs

pytestmark = pytest.mark.gpu

N = (1 << 21) + 37  # past the size from which tuples are computed


def _graph():
    """Hubs of chosen degrees among vertices of none to three, the ids of a hub and
    of what surrounds it close together."""
    rng = np.random.default_rng(0)
    u, v = [], []
    for block, deg in enumerate([7, 8, 9, 31, 32, 33, 64, 1000, 4095, 4096, 4097, 9000] * 2):
        at = 64 * 1300 * block
        for k, d in enumerate([deg] * (64 if deg < 100 else 3)):
            hub = at + 64 * (k // 2) + rng.integers(64)  # some share their step
            leaves = rng.choice(np.arange(at, at + 64 * 1300), d, replace=False)
            u.append(np.full(d, hub))
            v.append(leaves)
    w = rng.integers(0, N, 400_000)
    u.append(w)
    v.append(np.minimum(w + rng.integers(1, 200, w.size), N - 1))
    u, v = np.concatenate(u), np.concatenate(v)
    keep = u != v
    return graphs.from_edges(N, u[keep], v[keep])


@pytest.mark.parametrize("lanes", [0, 1])
def test_rows_of_all_lengths(lanes):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2204_02934_amd import _lib, api
    ctx = api.Context(0)
    ctx.set_option(_lib.MIS2_OPT_LANES_PER_ROW, lanes)
    rp, c = _graph()
    print("lanes", lanes, "n", N, "entries", c.size, flush=True)
    want, want_iters = oracle.mis2(rp, c, 3)
    status, _, iters = ctx.mis2(rp, c, 3)
    assert iters == want_iters and np.array_equal(status.cpu().numpy(), want)
    agg, n_agg = ctx.aggregate(rp, c, 3)
    want_agg, want_n = oracle.aggregate(rp, c, 3)
    assert n_agg == want_n and np.array_equal(agg.cpu().numpy(), want_agg)
