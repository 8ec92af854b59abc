"""Sorts whose workspace holds a part of the rows: windows of a few to many buckets,
which take narrower digits the more of them a window has."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.int32, torch.int64])
@pytest.mark.parametrize("per", [1, 20, 5000])
@pytest.mark.parametrize("n,part", [(3_000_000, 0.1), (23_412_627, 0.03), (23_412_627, 0.209), (23_412_627, 0.7)])
def test_sort(n, part, per, dtype):
    import paper_2602_21237_amd as tj
    tj.load()
    i = torch.iinfo(dtype)
    g = torch.Generator(device="cuda")
    g.manual_seed(per)
    values = torch.randint(i.min, i.max, (n // per,), device="cuda", generator=g, dtype=dtype)
    k = values[torch.randint(0, values.numel(), (n,), device="cuda", generator=g)] if per > 1 else values
    r = torch.arange(n, dtype=torch.int32, device="cuda")
    least, full = tj.tj.workspace_query(0, k.element_size(), n)
    ws = torch.empty(max(least, int(full * part)), dtype=torch.uint8, device="cuda")
    ko, ro = torch.empty_like(k), torch.empty_like(r)
    tj.sort(k, r, ko, ro, workspace=ws)
    want_k, want_r = torch.sort(k, stable=True)
    assert torch.equal(ko, want_k) and torch.equal(ro, want_r.to(torch.int32))
