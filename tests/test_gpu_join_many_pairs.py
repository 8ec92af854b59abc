"""Join blocks with many pairs a row, whose runs are written without staging:
fan-outs around the rule's edge, either side the smaller, runs with and without
a match in between, and a capacity that ends inside a run. Against the oracle."""
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


def check(tj, rk, sk, short=0):
    rng = np.random.default_rng(rk.size)
    rr, sr = rng.permutation(rk.size).astype(np.int32), rng.permutation(sk.size).astype(np.int32)
    xr, xs, cnt = oracle.join_pairs(rk, rr, sk, sr)
    assert tj.join_count(dev(rk), dev(sk)) == cnt
    out = torch.full((2, cnt + 64), -7, dtype=torch.int32, device="cuda")
    pr, ps = tj.join(dev(rk), dev(rr), dev(sk), dev(sr), capacity=cnt + 3, out_r=out[0], out_s=out[1])
    assert np.array_equal(pr.cpu().numpy(), xr) and np.array_equal(ps.cpu().numpy(), xs)
    assert bool((out[:, cnt:] == -7).all())
    if cnt > 100:  # the end of the outputs inside a run
        cap = cnt - 37
        out.fill_(-7)
        with pytest.raises(tj.TjError):
            tj.join(dev(rk), dev(rr), dev(sk), dev(sr), capacity=cap, out_r=out[0], out_s=out[1])
        assert bool((out[:, cap:] == -7).all())


@pytest.mark.parametrize("stride", [1, 7919, 1 << 44])
@pytest.mark.parametrize("a,b", [(5, 90), (6, 90), (7, 90), (7, 7), (10, 64), (10, 65), (48, 700), (49, 700), (20, 20), (33, 1)])
@pytest.mark.parametrize("swap", [False, True])
def test_even_fan_outs(tj, a, b, swap, stride):
    """`a` rows of the smaller side to `b` of the other, over one block and over many."""
    dtype = np.int64 if stride > 1 << 20 else np.int32
    for keys in (max(1, 6000 // (a + b)), 40_000 // (a + b) + 3):
        rng = np.random.default_rng(keys * a)
        few = rng.permutation(np.repeat(np.arange(keys), a)).astype(dtype) * dtype(stride)
        many = rng.permutation(np.repeat(np.arange(keys), b)).astype(dtype) * dtype(stride)
        check(tj, many, few) if swap else check(tj, few, many)


@pytest.mark.parametrize("dtype", [np.int32, np.int64])
@pytest.mark.parametrize("n_r,n_s", [(300, 7000), (7000, 300), (3000, 5000), (20_000, 90_000), (90_000, 20_000)])
def test_runs_of_all_sizes(tj, n_r, n_s, dtype):
    """Half of the keys on one side only; a few keys hold most rows."""
    rng = np.random.default_rng(n_r)
    keys = rng.integers(np.iinfo(dtype).min, np.iinfo(dtype).max, 3000, dtype=dtype)
    weight = 1.0 / np.arange(1, 2001) ** 1.1
    rk = rng.choice(keys[:2000], n_r, p=weight / weight.sum())
    sk = rng.choice(keys[1000:], n_s)
    hot = rng.integers(0, n_s, n_s // 2)
    sk[hot] = rng.choice(keys[:40], hot.size)
    check(tj, rk, sk)
