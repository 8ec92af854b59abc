"""Large calls over dense keys that one radix digit (9 bits) tells apart move their
rows once, on both sides of the spans that scatter whole lines."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N = 17_000_000


@pytest.mark.parametrize("dtype", [torch.int32, torch.int64])
@pytest.mark.parametrize("values", [2, 63, 64, 65, 256, 257, 512, 513])
def test_sort_passes(values, dtype):
    import paper_2602_21237_amd as tj
    tj.load()
    g = torch.Generator(device="cuda")
    g.manual_seed(values)
    k = torch.randint(0, values, (N,), device="cuda", generator=g, dtype=dtype) - 30
    r = torch.arange(N, dtype=torch.int32, device="cuda")
    ko, ro, st = tj.sort(k, r, stats=True)
    want_k, want_r = torch.sort(k, stable=True)
    assert torch.equal(ko, want_k)
    assert torch.equal(ro, want_r.to(torch.int32))
    assert values > 512 or st["passes"] == 1, st


@pytest.mark.parametrize("values", [63, 256, 459])
def test_join_passes(values):
    import paper_2602_21237_amd as tj
    tj.load()
    g = torch.Generator(device="cuda")
    g.manual_seed(values)
    rk = torch.randint(0, values, (N,), device="cuda", generator=g)
    sk = torch.arange(values, device="cuda")
    rr = torch.arange(N, dtype=torch.int32, device="cuda")
    sr = torch.arange(values, dtype=torch.int32, device="cuda") + 7
    r_rids, s_rids, st = tj.join(rk, rr, sk, sr, capacity=N, stats=True)
    assert torch.equal(torch.sort(r_rids).values, rr)
    assert torch.equal(rk[r_rids.to(torch.int64)] + 7, s_rids.to(torch.int64))
    assert st["passes"] == 1, st
