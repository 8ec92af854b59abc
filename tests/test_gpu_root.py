"""First passes that plan their digit on the device, against the oracle: key
spans on both sides of the widths where join keys narrow (2^41) and where one
scan block's 32 chunks of 9216 rows end, single keys, and a histogram digit
range sampled too narrow (the scatter then moves nothing and the pass repeats)."""
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


@pytest.mark.parametrize("bits", [1, 8, 31, 40, 41, 42, 63])
@pytest.mark.parametrize("n", [8193, 32 * 9216, 32 * 9216 + 1])
def test_sort_and_join_spans(tj, n, bits):
    rng = np.random.default_rng(n + bits)
    lo = -(1 << (bits - 1))
    rk = rng.integers(lo, lo + (1 << bits), n, dtype=np.int64)
    rk[:2] = lo, lo + (1 << bits) - 1
    if bits <= 8:  # few keys: an output of moderate size
        rk = np.where(np.arange(n) % 4096, lo - 1 - rng.integers(0, 1 << 40, n), rk)
    n_s = n // 2 + 7
    sk = np.where(rng.random(n_s) < 0.8, rk[rng.integers(0, n, n_s)], rng.integers(lo, lo + (1 << bits), n_s))
    rr, sr = rng.permutation(n).astype(np.int32), rng.permutation(n_s).astype(np.int32)
    ko, ro = tj.sort(dev(rk), dev(rr))
    ek, er = oracle.sort(rk, rr)
    assert np.array_equal(ko.cpu().numpy(), ek) and np.array_equal(ro.cpu().numpy(), er)
    xr, xs, cnt = oracle.join_pairs(rk, rr, sk, sr)
    pr, ps = tj.join(dev(rk), dev(rr), dev(sk), dev(sr))
    assert pr.numel() == cnt
    assert np.array_equal(pr.cpu().numpy(), xr) and np.array_equal(ps.cpu().numpy(), xs)


def test_single_key_and_sampled_miss(tj):
    k = np.full(20_000, -5, dtype=np.int64)
    r = np.arange(k.size, dtype=np.int32)[::-1].copy()
    ko, ro = tj.sort(dev(k), dev(r))
    assert np.array_equal(ko.cpu().numpy(), k) and np.array_equal(ro.cpu().numpy(), r)
    assert tj.join_count(dev(k), dev(k[:11_000])) == 20_000 * 11_000
    n = (1 << 22) + 5
    rng = np.random.default_rng(3)
    k = rng.integers(0, 1 << 30, n, dtype=np.int64)
    k[12_345] = 1 << 50   # between the sampled rows (every 4096th)
    r = rng.permutation(n).astype(np.int32)
    ko, ro = tj.sort(dev(k), dev(r))
    ek, er = oracle.sort(k, r)
    assert np.array_equal(ko.cpu().numpy(), ek) and np.array_equal(ro.cpu().numpy(), er)
