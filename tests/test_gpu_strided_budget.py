"""Few keys a power of two apart where the budget binds, so that every key is probed: one
radix digit tells them apart there too."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N = 17_000_000


@pytest.mark.parametrize("off", [(), (1, -1, 3)])
@pytest.mark.parametrize("dtype,stride", [(torch.int32, 12), (torch.int64, 40)])
@pytest.mark.parametrize("values", [1, 2, 50, 500])
def test_sort(values, dtype, stride, off):
    import paper_2602_21237_amd as tj
    tj.load()
    g = torch.Generator(device="cuda")
    g.manual_seed(values)
    k = torch.randint(0, values, (N,), device="cuda", generator=g, dtype=dtype) * (1 << stride) - 7
    for i, d in enumerate(off):
        k[N // 2 + 2 * i + 1] += d
    r = torch.arange(N, dtype=torch.int32, device="cuda")
    least, full = tj.tj.workspace_query(0, k.element_size(), N)
    ws = torch.empty(max(least, full // 3), dtype=torch.uint8, device="cuda")
    ko, ro = torch.empty_like(k), torch.empty_like(r)
    st = tj.sort(k, r, ko, ro, workspace=ws, stats=True)[2]
    want_k, want_r = torch.sort(k, stable=True)
    assert torch.equal(ko, want_k) and torch.equal(ro, want_r.to(torch.int32))
    assert off or st["passes"] <= 1, st
