"""The two kinds of compacting rounds: two and eight lanes a row with live bits,
sixteen without, and one lane a row on either side of the size from which the
large graphs' kernels run, against the CPU oracle."""
import numpy as np
import pytest

import oracle
from test_gpu_live_bits import N, _graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lanes,extra", [(2, 5), (8, 1), (16, 0), (1, -1), (1, 1)])
def test_aggregate(lanes, extra):
    from paper_2204_02934_amd import api
    rp, c = _graph(N + extra)
    print("lanes", lanes, "n", N + extra, "entries", c.size, flush=True)
    want, want_n = oracle.aggregate(rp, c, 3)
    for tail in (0, 1):
        agg, n_agg = api.Context(0, lanes=lanes, tail=tail).aggregate(rp, c, 3)
        assert n_agg == want_n and np.array_equal(agg.cpu().numpy(), want)
