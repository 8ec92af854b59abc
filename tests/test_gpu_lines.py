"""Passes of 2^24 rows and more, whose scatter writes whole lines: sorts and
joins against torch's stable sort, over key ranges with and without equal-part
digits, output columns that start inside a line, and forced re-ranking."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N = (1 << 24) + 12_345   # tiles, chunks and lines all end early


@pytest.fixture(scope="module")
def tj():
    import paper_2602_21237_amd as p
    p.load()
    return p


def gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def uniform64(n, g):
    hi = torch.randint(-(1 << 31), 1 << 31, (n,), device="cuda", generator=g)
    return (hi << 32) + torch.randint(0, 1 << 32, (n,), device="cuda", generator=g)


def sort_keys(kind, n, g):
    if kind == "i32":
        return torch.randint(-(1 << 31), 1 << 31, (n,), device="cuda", generator=g).to(torch.int32)
    if kind == "u64":
        return uniform64(n, g)
    if kind == "u40":
        return torch.randint(0, 1 << 40, (n,), device="cuda", generator=g)
    if kind == "u12":   # fewer key values than equal-part digits need
        return torch.randint(0, 3000, (n,), device="cuda", generator=g)
    if kind == "hot":   # a quarter of the rows in one key: a tile's lines belong to one digit
        k = uniform64(n, g)
        return torch.where(torch.rand(n, device="cuda", generator=g) < 0.25, torch.full_like(k, 77), k)
    return torch.exp(torch.randn(n, dtype=torch.float64, device="cuda", generator=g) * 2 + 30).to(torch.int64)


@pytest.mark.parametrize("force", [False, True])
@pytest.mark.parametrize("kind", ["i32", "u64", "u40", "u12", "hot", "lognormal"])
def test_sort(tj, kind, force):
    k = sort_keys(kind, N, gen(1))
    r = torch.randint(-(1 << 31), 1 << 31, (N,), device="cuda", generator=gen(2)).to(torch.int32)
    off = 5 if force else 0   # outputs at another place in their lines
    ko, ro = torch.empty(N + off, dtype=k.dtype, device="cuda")[off:], torch.empty(N + 3, dtype=r.dtype, device="cuda")[3:]
    tj.tj.debug_set_flags(tj.tj.TJ_DEBUG_FORCE_REORDER if force else 0)
    try:
        tj.sort(k, r, ko, ro)
    finally:
        tj.tj.debug_set_flags(0)
    ek, at = torch.sort(k, stable=True)
    assert torch.equal(ko, ek) and torch.equal(ro, r[at])


def pairs(r, s):
    """(R row, S row) of every match by key, R row, S row."""
    rk, ri = torch.sort(r, stable=True)
    sk, si = torch.sort(s, stable=True)
    lo = torch.searchsorted(sk, rk)
    n = torch.searchsorted(sk, rk, right=True) - lo
    i = torch.repeat_interleave(torch.arange(n.numel(), device="cuda"), n)
    j = torch.arange(i.numel(), device="cuda") - (torch.cumsum(n, 0) - n)[i] + lo[i]
    return ri[i], si[j]


@pytest.mark.parametrize("force", [False, True])
@pytest.mark.parametrize("kind", ["u40", "u64", "i32", "lognormal"])
def test_join(tj, kind, force):
    n_r = N // 4
    r = sort_keys(kind, n_r, gen(3))
    s = torch.cat([r[torch.randint(0, n_r, (N // 2,), device="cuda", generator=gen(4))],
                   sort_keys(kind, N - n_r - N // 2, gen(5))])
    er, es = pairs(r, s)
    rr, sr = (torch.arange(x.numel(), dtype=torch.int32, device="cuda") for x in (r, s))
    tj.tj.debug_set_flags(tj.tj.TJ_DEBUG_FORCE_REORDER if force else 0)
    try:
        c = tj.join_count(r, s)
        pr, ps = tj.join(r, rr, s, sr, capacity=c)
    finally:
        tj.tj.debug_set_flags(0)
    assert c == er.numel()
    assert torch.equal(pr.to(torch.int64), er) and torch.equal(ps.to(torch.int64), es)
