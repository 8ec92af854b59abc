"""Large calls over few keys a power of two apart: one radix digit tells them apart and
their rows move once; keys off the stride that the sample has not seen come out right."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N = 17_000_000


@pytest.fixture(scope="module")
def tj():
    import paper_2602_21237_amd as p
    p.load()
    return p


def column(values, stride, dtype, off=()):
    g = torch.Generator(device="cuda")
    g.manual_seed(values)
    k = torch.randint(0, values, (N,), device="cuda", generator=g, dtype=dtype) * (1 << stride)
    k -= 7 + torch.iinfo(dtype).max // 4
    for i, d in enumerate(off):
        k[N // 2 + 2 * i + 1] += d
    return k


@pytest.mark.parametrize("off", [(), (1, -1, 3)])
@pytest.mark.parametrize("dtype,stride", [(torch.int32, 1), (torch.int32, 21), (torch.int64, 40), (torch.int64, 53)])
@pytest.mark.parametrize("values", [2, 50, 200, 257, 500, 512])
def test_sort(tj, values, dtype, stride, off):
    k = column(values, stride, dtype, off)
    r = torch.arange(N, dtype=torch.int32, device="cuda")
    ko, ro, st = tj.sort(k, r, stats=True)
    want_k, want_r = torch.sort(k, stable=True)
    assert torch.equal(ko, want_k) and torch.equal(ro, want_r.to(torch.int32))
    assert off or st["passes"] == 1, st


@pytest.mark.parametrize("off", [(), (1, -1, 3)])
@pytest.mark.parametrize("values,stride", [(50, 33), (459, 9), (459, 33)])
def test_join(tj, values, stride, off):
    rk = column(values, stride, torch.int64, off)
    sk = (torch.arange(values, device="cuda") << stride) - 7 - torch.iinfo(torch.int64).max // 4
    rr = torch.arange(N, dtype=torch.int32, device="cuda")
    sr = torch.arange(values, dtype=torch.int32, device="cuda")
    r_rids, s_rids, st = tj.join(rk, rr, sk, sr, capacity=N, stats=True)
    r_rids = r_rids.to(torch.int64)
    keep = torch.ones(N, dtype=torch.bool, device="cuda")
    for i in range(len(off)):
        keep[N // 2 + 2 * i + 1] = False
    assert torch.equal(torch.sort(r_rids).values, torch.nonzero(keep).flatten())
    assert torch.equal(sk[s_rids.to(torch.int64)], rk[r_rids])
    assert off or st["passes"] == 1, st
