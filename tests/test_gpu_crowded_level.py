"""Large calls whose rows crowd one digit of the first level: the crowd takes full
radix digits, 512 values of it, a power of two apart, one level."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N = 17_000_000


def crowd(dtype, hot):
    i = torch.iinfo(dtype)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    k = torch.randint(0, 512, (N,), device="cuda", generator=g, dtype=dtype) * ((i.max >> 20) + 1)
    if hot:  # most rows of one key, which a pivot splits off
        k[torch.rand(N, device="cuda", generator=g) < 0.8] = 77
    k[0], k[-1] = i.min, i.max
    return k


@pytest.mark.parametrize("hot", [False, True])
@pytest.mark.parametrize("dtype", [torch.int32, torch.int64])
def test_sort(dtype, hot):
    import paper_2602_21237_amd as tj
    tj.load()
    k = crowd(dtype, hot)
    r = torch.arange(N, dtype=torch.int32, device="cuda")
    ko, ro, st = tj.sort(k, r, stats=True)
    want_k, want_r = torch.sort(k, stable=True)
    assert torch.equal(ko, want_k) and torch.equal(ro, want_r.to(torch.int32))
    assert hot or st["passes"] == 2, st


@pytest.mark.parametrize("hot", [False, True])
@pytest.mark.parametrize("dtype", [torch.int32, torch.int64])
def test_join(dtype, hot):
    import paper_2602_21237_amd as tj
    tj.load()
    k = crowd(dtype, hot)
    few = torch.unique(k)
    few = few[few != 77].contiguous()
    at = torch.nonzero(k != 77).flatten()
    r = torch.arange(N, dtype=torch.int32, device="cuda")
    pr, ps = tj.join(k, r, few, r[:few.numel()], capacity=N)
    pr = pr.to(torch.int64)
    assert torch.equal(torch.sort(pr).values, at)
    assert torch.equal(few[ps.to(torch.int64)], k[pr])
