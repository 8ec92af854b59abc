"""Inputs of one block (at most 8192 rows): the single-launch sort and join
against the oracle, at the edges of their block shapes and one row beyond."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

I64 = np.iinfo(np.int64)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.fixture(scope="module")
def tj():
    import paper_2602_21237_amd as p
    p.load()
    return p


def keys_of(kind, n, rng):
    if kind == "i32":
        return rng.integers(-(1 << 31), 1 << 31, n).astype(np.int32)
    if kind == "i64":
        k = rng.integers(I64.min, I64.max, n, dtype=np.int64)
        k[:2] = (I64.max, I64.min)[:k[:2].size]
        return k
    if kind == "equal":
        return np.full(n, I64.min, dtype=np.int64)
    return rng.integers(-20, 20, n).astype(np.int64)  # many rows a key


@pytest.mark.parametrize("kind", ["i32", "i64", "few", "equal"])
@pytest.mark.parametrize("n", [1, 2, 255, 256, 1023, 1024, 1025, 4095, 4096, 4097, 8191, 8192, 8193])
def test_small_sort(tj, n, kind):
    rng = np.random.default_rng(n)
    k = keys_of(kind, n, rng)
    r = rng.integers(-(1 << 31), 1 << 31, n).astype(np.int32)
    ko, ro, st = tj.sort(dev(k), dev(r), stats=True)
    ek, er = oracle.sort(k, r)
    assert np.array_equal(ko.cpu().numpy(), ek) and np.array_equal(ro.cpu().numpy(), er)
    assert st["passes"] == (1 if n > 8192 else 0), st


@pytest.mark.parametrize("force", [False, True])
@pytest.mark.parametrize("kind", ["i32", "i64", "few"])
@pytest.mark.parametrize("n_r,n_s", [(1, 1), (1, 1023), (512, 512), (513, 512), (4000, 96), (97, 4000), (4096, 4096),
                                     (8191, 1), (1, 8191), (4097, 4096)])
def test_small_join(tj, n_r, n_s, kind, force):
    rng = np.random.default_rng(n_r * 7 + n_s)
    rk = keys_of(kind, n_r, rng)
    sk = np.where(rng.random(n_s) < 0.7, rng.choice(rk, n_s), keys_of(kind, n_s, rng)).astype(rk.dtype)
    rr, sr = rng.permutation(n_r).astype(np.int32), rng.permutation(n_s).astype(np.int32)
    xr, xs, cnt = oracle.join_pairs(rk, rr, sk, sr)
    tj.tj.debug_set_flags(tj.tj.TJ_DEBUG_FORCE_REORDER if force else 0)
    try:
        assert tj.join_count(dev(rk), dev(sk)) == cnt
        pr, ps = tj.join(dev(rk), dev(rr), dev(sk), dev(sr), capacity=cnt + 3)
    finally:
        tj.tj.debug_set_flags(0)
    assert np.array_equal(pr.cpu().numpy(), xr) and np.array_equal(ps.cpu().numpy(), xs)
    if cnt:  # one pair short: the count, and nothing past the end
        out = torch.full((2, cnt), -7, dtype=torch.int32, device="cuda")
        with pytest.raises(tj.TjError):
            tj.join(dev(rk), dev(rr), dev(sk), dev(sr), capacity=cnt - 1, out_r=out[0], out_s=out[1])
        assert int(out[0, -1]) == -7 and int(out[1, -1]) == -7
