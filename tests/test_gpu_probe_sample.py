"""The sampled range of a large call: read once for periodic keys and for a side of
few rows (a row outside it costs a second look at every key)."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N = 17_000_000


@pytest.fixture
def tj():
    import paper_2602_21237_amd as p
    p.load()
    p.tj.timing(True)
    yield p
    p.tj.timing(False)


def rows(n):
    return torch.arange(n, dtype=torch.int32, device="cuda")


@pytest.mark.parametrize("n", [1 << 22, N])
@pytest.mark.parametrize("period", [4096, 12288])
def test_periodic_keys(tj, period, n):
    k = torch.arange(n, device="cuda") % period - 5
    ko, ro = tj.sort(k, rows(n))
    d = tj.tj.timing_read()
    want_k, want_r = torch.sort(k, stable=True)
    assert torch.equal(ko, want_k) and torch.equal(ro, want_r.to(torch.int32))
    assert d["probe"]["launches"] == 1, d


@pytest.mark.parametrize("few_first", [True, False])
@pytest.mark.parametrize("n", [1, 8191, 8193, 400_000])
def test_few_rows_of_a_side(tj, n, few_first):
    # one row in 8 of the short side spans 8 times the rest, none where 4096 divides the row
    far = (rows(n) % 8 == 3).to(torch.int64)
    few = rows(n).to(torch.int64) % 1000 + far * (rows(n).to(torch.int64) * 7919 % 8000 - 4000)
    many = torch.arange(N, device="cuda") % 1000
    cols = [few, rows(n), many, rows(N)]
    a = cols if few_first else cols[2:] + cols[:2]
    cnt = tj.join_count(a[0], a[2])
    d = tj.tj.timing_read()
    h = torch.bincount(many, minlength=8192).cpu()
    inside = few[(few >= 0) & (few < 1000)].cpu()
    assert cnt == int(h[inside].sum())
    assert d["probe"]["launches"] == 1, d
