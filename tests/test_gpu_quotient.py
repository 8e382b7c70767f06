"""GPU parity of the quotient graph at the limits of its row paths: the distinct
ids and candidates a lane group, a wavefront and a workgroup take, rows of the
bitmap slots beyond their number, and a spare buffer with no room left.  The
rows are hubs with a chosen number of leaves; the oracle's quotient decides."""
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


def _hubs(sizes, leaves, alone=0, leaf_labels=None, seed=0):
    """Hub k joined to sizes[k] random leaves; every hub and every lone vertex an
    aggregate of its own, and so every leaf unless leaf_labels groups them."""
    rng = np.random.default_rng(seed)
    h = len(sizes)
    u = np.repeat(np.arange(h), sizes)
    v = h + np.concatenate([rng.choice(leaves, s, replace=False) for s in sizes])
    rp, c = graphs.from_edges(h + leaves + alone, u, v)
    lab = np.arange(h + leaves + alone)
    if leaf_labels:
        lab[h:h + leaves] = h + np.arange(leaves) % leaf_labels
        lab[h + leaves:] -= leaves - leaf_labels
    perm = rng.permutation(int(lab.max()) + 1)  # ids in no particular order
    return rp, c, perm[lab].astype(np.int32), int(lab.max()) + 1


def _random(n, deg, n_agg, seed=0):
    rp, c = graphs.random_regular_ish(n, deg, seed=seed)
    return rp, c, np.random.default_rng(seed).permutation(np.arange(n) % n_agg).astype(np.int32), n_agg


CASES = {
    # a 16-lane group: fewer than 96 distinct ids, at most 512 candidates
    "group16_ids": lambda: _hubs([94, 95, 96, 97], 300),
    "group16_candidates": lambda: _hubs([511, 512, 513], 600, leaf_labels=20),
    # a wavefront with the small set (more than 256 candidates a row on average)
    "group64_ids": lambda: _random(4000, 60, 159),
    "group64_over": lambda: _random(4000, 60, 163),
    # more than 393216 coarse ids: 1024-slot sets, then workgroups in windows
    "set_ids": lambda: _hubs([95, 96, 766, 767, 768, 769, 8192, 8193], 9000, alone=395_000),
    "set_candidates": lambda: _hubs([8192, 8193], 9000, alone=395_000, leaf_labels=100),
    "set_no_room": lambda: _hubs([700] * 2600, 9000, alone=395_000),
    # bitmap slots: rows of more than 16384 candidates, more rows than slots
    "slots": lambda: _hubs([16383, 16384, 16385] + [16390] * 11, 16400),
    "slots_few_ids": lambda: _hubs([16384, 16385, 20000], 20000, leaf_labels=3),
    # one aggregate, no neighbours
    "one": lambda: _random(3000, 40, 1),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_quotient_row_paths(ctx, name):
    rp, c, lab, n_agg = CASES[name]()
    crow, ccol = ctx.quotient(rp, c, lab, n_agg)
    orow, ocol = oracle.quotient(rp, c, lab, n_agg)
    assert np.array_equal(crow.cpu().numpy(), orow)
    assert np.array_equal(ccol.cpu().numpy(), ocol)
