"""GPU parity of phase 3's rows past the register path: rows of 32 / 33, 64 / 65,
128 / 129 and 512 / 513 entries, rows of one aggregate or of many, and rows with
more aggregates than the LDS map holds at once, against the oracle's labels."""
import numpy as np
import pytest

import oracle
from paper_2204_02934_amd import graphs

pytestmark = pytest.mark.gpu


def _late(rows, seed=0):
    """Components with one vertex each that only phase 3 can label.  rows[k] lists
    how many of that vertex's neighbours belong to each of its aggregates: root i
    has rows[k][i] leaves, all joined to the vertex.  The ids of the smallest
    round-0 tuples go to the roots, which so win round 0 and take their leaves;
    the vertex is left alone."""
    n = sum(1 + len(r) + sum(r) for r in rows)
    b = oracle.id_bits(n)
    t = np.array([oracle.pack(oracle.hash_priority(seed, 0, v), v, b) for v in range(n)], np.uint64)
    order = np.argsort(t, kind="stable")
    n_roots = sum(len(r) for r in rows)
    roots, rest = order[:n_roots], np.random.default_rng(seed).permutation(order[n_roots:])
    u, v, i, j = [], [], 0, 0
    for r in rows:
        r = np.asarray(r)
        hub, leaves = rest[j], rest[j + 1:j + 1 + r.sum()]
        u += [np.repeat(roots[i:i + r.size], r), np.full(leaves.size, hub)]
        v += [leaves, leaves]
        i, j = i + r.size, j + 1 + leaves.size
    return graphs.from_edges(n, np.concatenate(u), np.concatenate(v))


def _split(total, most, seed):
    """Aggregates of 1 .. most neighbours each that make a row of `total`."""
    rng, out = np.random.default_rng(seed), []
    while sum(out) < total:
        out.append(int(min(rng.integers(1, most + 1), total - sum(out))))
    return out


CASES = {
    "short": lambda: _late([_split(t, 3, t) for t in (1, 2, 31, 32, 33, 34)]),
    "mid": lambda: _late([_split(t, 5, t) for t in (63, 64, 65, 127, 128, 129, 200)]),
    "one_id": lambda: _late([[t] for t in (33, 64, 65, 512, 513, 2100)]),
    "mid_long": lambda: _late([_split(t, 4, t) for t in (511, 512, 513, 514, 1500)]),
    # more distinct aggregates than the LDS map takes at once: 2 and 5 classes
    "two_classes": lambda: _late([[1] * 4096, [1] * 4096 + [2], [3] + [1] * 6000]),
    "many_classes": lambda: _late([[1] * 9000 + [2] + [1] * 9000]),
    "elasticity": lambda: graphs.elasticity3d(14, 13, 15),
    "chunglu": lambda: graphs.chung_lu(60_000, 24.0, 2.0, 9000, seed=3),
}


@pytest.mark.parametrize("lanes", [0, 1, 4, 16, 64])
@pytest.mark.parametrize("name", sorted(CASES))
def test_aggregate(name, lanes):
    from paper_2204_02934_amd import api
    rp, c = CASES[name]()
    ctx = api.Context(0, lanes=lanes)
    want, n_agg = oracle.aggregate(rp, c, 0)
    got, na = ctx.aggregate(rp, c, 0)
    assert na == n_agg
    assert np.array_equal(got.cpu().numpy(), want)
