"""Large inputs whose sampled keys (every 4096th row) are all one key, though
others are not: the range is not the sample's. Against the oracle."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N = 1 << 22  # rows from which the first digit's range is sampled


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.fixture(scope="module")
def tj():
    import paper_2602_21237_amd as p
    p.load()
    return p


def column(kind, n, dtype):
    if kind == "one row":
        k = np.full(n, -3, dtype=dtype)
        k[n // 2 + 1] = np.iinfo(dtype).max
    elif kind == "rare":  # one row in 5000
        k = np.zeros(n, dtype=dtype)
        at = np.arange(7, n, 5000)
        at = at[at % 4096 != 0]
        k[at] = np.random.default_rng(n).integers(-1000, 1000, at.size)
    else:  # a period of the sample's step
        k = (np.arange(n) % 4096 - 9).astype(dtype)
    assert np.unique(k[::4096]).size == 1 and np.unique(k).size > 1
    return k


@pytest.mark.parametrize("dtype", [np.int32, np.int64])
@pytest.mark.parametrize("kind", ["one row", "rare", "period"])
@pytest.mark.parametrize("n", [N, N + 4097])
def test_sort(tj, n, kind, dtype):
    k = column(kind, n, dtype)
    r = np.random.default_rng(n).permutation(n).astype(np.int32)
    ek, er = oracle.sort(k, r)
    for part in ("radix", "auto"):
        ko, ro = tj.sort(dev(k), dev(r), partitioner=part)
        assert np.array_equal(ko.cpu().numpy(), ek) and np.array_equal(ro.cpu().numpy(), er), part


@pytest.mark.parametrize("dtype", [np.int32, np.int64])
@pytest.mark.parametrize("kind", ["one row", "rare", "period"])
@pytest.mark.parametrize("n_r,n_s", [(3, N + 4097), (N + 1, 3)])
def test_join(tj, n_r, n_s, kind, dtype):
    # (the sample takes the last row too: each side ends with the sampled key)
    big = column(kind, max(n_r, n_s), dtype)
    rest = np.unique(big)
    short = np.array([big[0], rest[rest != big[0]][-1], big[0]], dtype=dtype)
    assert big[-1] == big[0]
    rk, sk = (short, big) if n_r < n_s else (big, short)
    rng = np.random.default_rng(n_r + n_s)
    rr, sr = rng.permutation(rk.size).astype(np.int32), rng.permutation(sk.size).astype(np.int32)
    xr, xs, cnt = oracle.join_pairs(rk, rr, sk, sr)
    assert tj.join_count(dev(rk), dev(sk)) == cnt
    pr, ps = tj.join(dev(rk), dev(rr), dev(sk), dev(sr), capacity=cnt + 3)
    assert np.array_equal(pr.cpu().numpy(), xr) and np.array_equal(ps.cpu().numpy(), xs)
