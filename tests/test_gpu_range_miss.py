"""Rows outside the sampled range of a large call: the pass starts again with the range
that its histogram saw, without another probe."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture
def tj():
    import paper_2602_21237_amd as p
    p.load()
    p.tj.timing(True)
    yield p
    p.tj.timing(False)


def column(n, dtype, where):
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    k = torch.randint(-5000, 5000, (n,), device="cuda", generator=g, dtype=dtype)
    i = torch.iinfo(dtype)
    if "low" in where:
        k[n // 2 + 1] = i.min
    if "high" in where:
        k[n // 2 + 3] = i.max
    if "near" in where:
        k[n // 2 + 5] = 9000
    return k


@pytest.mark.parametrize("part", ["radix", "auto"])
@pytest.mark.parametrize("where", ["low", "high", "low high", "near"])
@pytest.mark.parametrize("dtype", [torch.int32, torch.int64])
@pytest.mark.parametrize("n", [(1 << 22) + 1, 17_000_000])
def test_sort(tj, n, dtype, where, part):
    k = column(n, dtype, where)
    r = torch.arange(n, dtype=torch.int32, device="cuda")
    ko, ro = tj.sort(k, r, partitioner=part)
    d = tj.tj.timing_read()
    want_k, want_r = torch.sort(k, stable=True)
    assert torch.equal(ko, want_k) and torch.equal(ro, want_r.to(torch.int32))
    assert part != "radix" or d["probe"]["launches"] == 1, d


@pytest.mark.parametrize("side", [0, 1])
@pytest.mark.parametrize("where", ["low high", "near"])
@pytest.mark.parametrize("dtype", [torch.int32, torch.int64])
def test_join(tj, dtype, where, side):
    n = 17_000_000
    big = column(n, dtype, where)
    edge = torch.iinfo(dtype)
    few = torch.tensor([edge.min, 3, 9000, edge.max], device="cuda", dtype=dtype)
    rows = lambda m: torch.arange(m, dtype=torch.int32, device="cuda")
    a = [big, rows(n), few, rows(4)]
    a = a[2:] + a[:2] if side else a
    pairs = int(torch.isin(big, few).sum())
    pr, ps = tj.join(*a, capacity=pairs + 1)
    d = tj.tj.timing_read()
    if side:
        pr, ps = ps, pr
    at = torch.nonzero(torch.isin(big, few)).flatten()
    order = torch.argsort(pr)
    assert torch.equal(pr[order].to(torch.int64), at)
    assert torch.equal(few[ps[order].to(torch.int64)], big[at])
    if where != "near":  # (the short side holds the extremes; a row between them misses nothing)
        few2 = few[1:3].contiguous()
        a[0 if side else 2], a[1 if side else 3] = few2, rows(2)
        tj.tj.timing(False)
        tj.tj.timing(True)  # (off and on clears the counters)
        assert tj.join_count(a[0], a[2]) == int(torch.isin(big, few2).sum())
        d = tj.tj.timing_read()
    assert d["probe"]["launches"] == 1, d
