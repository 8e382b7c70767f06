"""GPU parity of the one-workgroup form of small graphs on its longer rows, each
graph asserted to be inside (or just past) its limits: hubs that phase 3 leaves to
the workgroup, coupled to many aggregates with ties in coupling and in size; roots
of either phase with more than 128 neighbours to take; exactly as many entries as
it holds and two more.  The launched form of the same graphs, and of every graph of
test_gpu_small.py, is compared with the oracle too."""
import numpy as np
import pytest

import oracle
import test_gpu_small
from paper_2204_02934_amd import graphs
from test_gpu_phase3 import _late, _split

pytestmark = pytest.mark.gpu


def _edges(n, m, seed):
    """A random graph of exactly m edges."""
    key = np.random.default_rng(seed).choice(n * (n - 1) // 2, m, replace=False)
    u, v = np.triu_indices(n, 1)
    return graphs.from_edges(n, u[key], v[key])


def _order(n, seed=0):
    """Vertices by their round-0 tuple."""
    b = oracle.id_bits(n)
    t = np.array([oracle.pack(oracle.hash_priority(seed, 0, v), v, b) for v in range(n)], np.uint64)
    return np.argsort(t, kind="stable")


def _second_roots(leaves):
    """Components with a root, its neighbour b, and a hub and leaves joined to b and
    to each other: only b is taken in phase 1, and the hub, first among the others,
    takes its leaves in phase 2."""
    n = sum(3 + k for k in leaves)
    order, u, v, at = _order(n), [], [], 2 * len(leaves)
    for i, k in enumerate(leaves):
        root, hub = order[i], order[len(leaves) + i]
        b, own = order[at], order[at + 1:at + 1 + k]
        at += 1 + k
        u += [[root, b], np.full(k, b), np.full(k, hub)]
        v += [[b, hub], own, own]
    return graphs.from_edges(n, np.concatenate(u), np.concatenate(v))


def _first_roots(leaves):
    """Stars whose centres come first."""
    order, at = _order(sum(leaves) + len(leaves)), len(leaves)
    own = [order[at + sum(leaves[:i]):at + sum(leaves[:i + 1])] for i in range(len(leaves))]
    u = [np.full(k, order[i]) for i, k in enumerate(leaves)]
    return graphs.from_edges(order.size, np.concatenate(u), np.concatenate(own))


IN = {
    # the workgroup's rows (more than 512 entries): one, and several
    "hub600": lambda: _late([_split(600, 5, 1)]),
    "hub2400": lambda: _late([[1, 2, 3] * 300 + [3] * 200]),
    "hubs": lambda: _late([_split(t, 4, t) for t in (513, 514, 700)]),
    "ties": lambda: _late([[2] * 300 + [1] * 40, [1] * 513, [3] * 180 + [2] * 20]),
    "few": lambda: _late([[520], [260, 260], [200, 200, 200], [300, 299]]),
    # a wavefront's
    "mid": lambda: _late([_split(t, 3, t) for t in (32, 33, 64, 65, 128, 129, 511, 512)]),
    "second_roots": lambda: _second_roots([2, 127, 128, 129, 200, 1500]),
    "first_roots": lambda: _first_roots([127, 128, 129, 130, 2000]),
    "dense": lambda: graphs.complete(150),
    "z32768": lambda: _edges(4096, 16384, 5),
    "z32768_few": lambda: _edges(400, 16384, 6),
}
PAST = {"z32770": lambda: _edges(4096, 16385, 7), "n4097": lambda: _edges(4097, 9000, 8)}


def _check(ctx, rp, c, seed):
    want, rounds = oracle.mis2(rp, c, seed)
    st, nr, it = ctx.mis2(rp, c, seed)
    assert np.array_equal(st.cpu().numpy(), want) and (nr, it) == (int(want.sum()), rounds)
    lab, n_agg = oracle.aggregate(rp, c, seed)
    got, na, roots = ctx.aggregate(rp, c, seed, want_roots=True)
    assert na == n_agg and np.array_equal(got.cpu().numpy(), lab)
    return roots.cpu().numpy()


@pytest.mark.parametrize("name", sorted(IN) + sorted(PAST))
def test_rows(name):
    from paper_2204_02934_amd import api
    rp, c = (IN.get(name) or PAST[name])()
    assert (rp.size - 1 <= 4096 and c.size <= 32768) == (name in IN), (rp.size - 1, c.size)
    for seed in (0, 4):
        ctx = api.Context(0)
        roots = _check(ctx, rp, c, seed)
        whole = [r["round"] == 0 for r in ctx.last_sweeps() if r["kind"] == 3]
        assert (whole == [True, True]) == (name in IN)
        other = _check(api.Context(0, autotune=False), rp, c, seed)
        assert np.array_equal(roots, other)
        if seed == 0 and name in ("second_roots", "first_roots"):
            # (a second root's row holds b as well)
            mark, row = (2, 129) if name == "second_roots" else (1, 128)
            assert (np.diff(rp)[roots == mark] > row).sum() == 3


@pytest.mark.parametrize("name", sorted(test_gpu_small.CASES))
def test_launched(name):
    from paper_2204_02934_amd import api
    rp, c = test_gpu_small.CASES[name]()
    for seed in (0, 3):
        _check(api.Context(0, autotune=False), rp, c, seed)
