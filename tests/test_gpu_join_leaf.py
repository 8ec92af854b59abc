"""The LDS block of the join at the edges of its ways: runs of as many S rows as
are ranked by looking at all of them and one more, as many R rows in one bin as
the binned way takes and one more, R sides around what the pool holds, and the
largest key of the whole type beside the table's padding. Inputs of one block
and of several; values and order are exact."""
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


def check(tj, rk, sk, rng):
    rr = rng.integers(-(1 << 31), 1 << 31, rk.size).astype(np.int32)
    sr = rng.integers(-(1 << 31), 1 << 31, sk.size).astype(np.int32)
    xr, xs, cnt = oracle.join_pairs(rk, rr, sk, sr)
    assert tj.join_count(dev(rk), dev(sk)) == cnt
    pr, ps = tj.join(dev(rk), dev(rr), dev(sk), dev(sr), capacity=cnt + 1)
    assert np.array_equal(pr.cpu().numpy(), xr) and np.array_equal(ps.cpu().numpy(), xs)


@pytest.mark.parametrize("others", [500, 9000])
@pytest.mark.parametrize("dtype", [np.int32, np.int64])
@pytest.mark.parametrize("a,b", [(1, 31), (2, 32), (1, 33), (3, 3000), (47, 100), (48, 129), (49, 128), (700, 3), (32, 3), (33, 2)])
def test_runs(tj, a, b, dtype, others):
    """A run of a R and b S rows between others, and a second one of S rows beside it."""
    rng = np.random.default_rng(a * 1000 + b)
    info = np.iinfo(dtype)
    rk = rng.integers(info.min, info.max, others // 4, dtype=dtype)
    sk = np.concatenate([rng.choice(rk, others // 2), rng.integers(info.min, info.max, others // 4, dtype=dtype)])
    key = dtype(info.max // 3)
    rk = np.concatenate([rk, np.full(a, key, dtype), np.array([key + 1], dtype)])
    sk = np.concatenate([sk, np.full(b, key, dtype), np.full(b // 2 + 1, key + 1, dtype)])
    check(tj, rng.permutation(rk), rng.permutation(sk), rng)


@pytest.mark.parametrize("dtype", [np.int32, np.int64])
@pytest.mark.parametrize("n_r,n_s", [(4095, 4096), (5300, 90), (5400, 90), (6100, 90), (8100, 90), (8192, 0), (0, 8192),
                                     (6000, 60000), (60000, 6000)])
def test_sides(tj, n_r, n_s, dtype):
    """R sides around the pool's size, and one empty side; the type's largest and smallest keys on both sides."""
    rng = np.random.default_rng(n_r + n_s)
    info = np.iinfo(dtype)
    ends = np.array([info.max, info.min, info.max, info.max - 1], dtype)
    rk = rng.integers(info.min, info.max, n_r, dtype=dtype)
    sk = rng.integers(info.min, info.max, n_s, dtype=dtype)
    if n_r and n_s:
        sk[: n_s // 2] = rng.choice(rk, n_s // 2)
        rk[-4:], sk[-4:] = ends, ends
    check(tj, rk, sk, rng)
