"""Prefix sums of more than 2^29 values, whose threads add up in 64 bits: the
quotient graph of a sparse graph under the identity labelling is the graph itself.
(About 50 GB of device memory.)"""
import pytest

pytestmark = pytest.mark.gpu


def test_identity_quotient():
    import torch
    from paper_2204_02934_amd import api
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 100 GB of free device memory")
    n = (1 << 29) + 5
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    u = 2 * torch.unique(torch.randint(0, n // 2, (500_000,), device="cuda", generator=g))
    u = torch.cat([u, torch.tensor([n - 3], device="cuda")])  # n is odd: n - 3 is even
    u = torch.unique(u)
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rp[u + 1] = 1
    rp[u + 2] = 1
    torch.cumsum(rp, 0, out=rp)
    col = torch.stack([u + 1, u], 1).flatten().to(torch.int32)
    assert int(rp[-1].item()) == col.numel()
    agg = torch.arange(n, dtype=torch.int32, device="cuda")
    print("n", n, "entries", col.numel(), flush=True)
    crow, ccol = api.Context(0).quotient(rp, col, agg, n, nnz=col.numel())
    assert torch.equal(crow, rp) and torch.equal(ccol, col)
