"""Learned joins whose second pass narrows the keys of segments that span less
than 2^32 ordinals: their neighbouring buckets share leaves."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("step,share", [(8, True), (1 << 33, False)])
def test_leaves_are_shared(step, share):
    """R: 2^27 keys `step` apart, with gaps; S: as many rows on them. step 2^33: the
    buckets span more than 2^32 ordinals, and each keeps its own."""
    import paper_2602_21237_amd as tj
    tj.load()
    n = 1 << 27
    g = torch.Generator(device="cuda")
    g.manual_seed(step % 1000)
    gap = torch.randint(0, 5, (n,), device="cuda", generator=g)
    rk = (torch.cumsum(gap, 0) + torch.arange(n, device="cuda")) * step
    del gap
    at = torch.randint(0, n, (n,), device="cuda", generator=g)
    sk = rk[at]
    ids = torch.arange(n, dtype=torch.int32, device="cuda")
    cnt, st = tj.join_count(rk, sk, stats=True, partitioner="learned")
    assert cnt == n and st["learned"] == 1
    pr, ps, st = tj.join(rk, ids, sk, ids, capacity=n, stats=True, partitioner="learned")
    a, b = pr.to(torch.int64), ps.to(torch.int64)
    assert pr.numel() == n and torch.equal(rk[a], sk[b])
    assert bool(((a[1:] > a[:-1]) | ((a[1:] == a[:-1]) & (b[1:] > b[:-1]))).all())  # canonical, so each S row once
    rows_a_leaf = 2 * n / st["leaves"]
    assert rows_a_leaf > (5500 if share else 2500), st
