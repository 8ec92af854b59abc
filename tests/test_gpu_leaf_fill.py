"""Large sorts with several rows a key: the spread of the first level's buckets
tells how full the second level's may be planned, so that none takes a third."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per", [1, 8, 32])
def test_two_levels_do(per):
    import paper_2602_21237_amd as tj
    tj.load()
    n = 90_000_000
    g = torch.Generator(device="cuda")
    g.manual_seed(per)
    values = torch.randint(-(1 << 62), 1 << 62, (n // per,), device="cuda", generator=g)
    k = values[torch.randint(0, values.numel(), (n,), device="cuda", generator=g)] if per > 1 else values
    r = torch.arange(n, dtype=torch.int32, device="cuda")
    ko, ro, st = tj.sort(k, r, stats=True)
    assert bool((ko[1:] >= ko[:-1]).all())
    at = ro.to(torch.int64)
    assert torch.equal(k[at], ko)  # every row with its key
    assert bool(((at[1:] > at[:-1]) | (ko[1:] > ko[:-1])).all())  # stable, so each row once
    assert int(at.sum()) == n * (n - 1) // 2
    assert st["passes"] == 2, st
