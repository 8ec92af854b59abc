"""Inputs of one key (and of one key but for one row) beyond one block: against
the oracle, and no pass moves a row of the former."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.fixture(scope="module")
def tj():
    import paper_2602_21237_amd as p
    p.load()
    return p


def column(n, dtype, odd_at):
    k = np.full(n, np.iinfo(dtype).min if n % 2 else -3, dtype=dtype)
    if odd_at is not None:
        k[odd_at] = np.iinfo(dtype).max
    return k


@pytest.mark.parametrize("dtype", [np.int32, np.int64])
@pytest.mark.parametrize("odd", [False, True])
@pytest.mark.parametrize("n", [8193, 100_003, (1 << 22) - 1, 1 << 22, (1 << 22) + 5])
def test_sort_of_one_key(tj, n, odd, dtype):
    k = column(n, dtype, n // 2 + 1 if odd else None)
    r = np.random.default_rng(n).permutation(n).astype(np.int32)
    ko, ro, st = tj.sort(dev(k), dev(r), stats=True)
    ek, er = oracle.sort(k, r)
    assert np.array_equal(ko.cpu().numpy(), ek) and np.array_equal(ro.cpu().numpy(), er)
    if not odd:
        assert st["single_key"] == 1 and st["leaves"] == 0 and st["bytes_written"] == n * (k.itemsize + 4), st


@pytest.mark.parametrize("dtype", [np.int32, np.int64])
@pytest.mark.parametrize("odd", [False, True])
@pytest.mark.parametrize("n_r,n_s", [(1, 8192), (8192, 1), (5000, 4000), (300, 100_001), (3, 1 << 22)])
def test_join_of_one_key(tj, n_r, n_s, odd, dtype):
    rk, sk = column(n_r, dtype, None), column(n_s, dtype, n_s // 3 if odd else None)
    sk[sk != np.iinfo(dtype).max] = rk[0]
    rng = np.random.default_rng(n_r + n_s)
    rr, sr = rng.permutation(n_r).astype(np.int32), rng.permutation(n_s).astype(np.int32)
    xr, xs, cnt = oracle.join_pairs(rk, rr, sk, sr)
    got, st = tj.join_count(dev(rk), dev(sk), stats=True)
    assert got == cnt
    pr, ps = tj.join(dev(rk), dev(rr), dev(sk), dev(sr), capacity=cnt + 3)
    assert np.array_equal(pr.cpu().numpy(), xr) and np.array_equal(ps.cpu().numpy(), xs)
    if not odd:
        assert st["single_key"] == 1 and st["bytes_written"] == 0, st
        out = torch.full((2, cnt), -7, dtype=torch.int32, device="cuda")
        with pytest.raises(tj.TjError):
            tj.join(dev(rk), dev(rr), dev(sk), dev(sr), capacity=cnt - 1, out_r=out[0], out_s=out[1])
        assert int(out[0, -1]) == -7 and int(out[1, -1]) == -7


@pytest.mark.parametrize("n_r,n_s", [(9000, 100), (100_000, 50_000)])
def test_join_without_a_match(tj, n_r, n_s):
    """Two keys, one a side: the host's list of leaves is empty."""
    rk, sk = np.full(n_r, 7, np.int64), np.full(n_s, 8, np.int64)
    assert tj.join_count(dev(rk), dev(sk)) == 0
    ids = torch.arange(n_r, dtype=torch.int32, device="cuda")
    pr, ps = tj.join(dev(rk), ids, dev(sk), ids[:n_s].contiguous(), capacity=4)
    assert pr.numel() == 0 and ps.numel() == 0
