"""Single-key buckets at the edges of a block's stretch: rows copied to the sort's
output and pairs of cross products, in units of odd lengths beside one another,
from less than one block's rows to several blocks for every CU."""
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


@pytest.mark.parametrize("dtype", [np.int32, np.int64])
@pytest.mark.parametrize("hot", [(8193,), (8193, 10240, 10241), (9001, 8200, 50_003, 300_001), (5_000_001,)])
def test_copies(tj, hot, dtype):
    rng = np.random.default_rng(len(hot))
    info = np.iinfo(dtype)
    keys = [np.full(c, info.max // 3 + 7 * i, dtype) for i, c in enumerate(hot)]
    k = rng.permutation(np.concatenate(keys + [rng.integers(info.min, info.max, 20_000, dtype=dtype)]))
    r = rng.integers(-(1 << 31), 1 << 31, k.size).astype(np.int32)
    ko, ro = tj.sort(dev(k), dev(r))
    o = np.argsort(k, kind="stable")
    assert np.array_equal(ko.cpu().numpy(), k[o]) and np.array_equal(ro.cpu().numpy(), r[o])


@pytest.mark.parametrize("a,b", [(1, 9001), (9001, 1), (3, 8200), (700, 9003), (2, 3_000_001)])
def test_crosses(tj, a, b):
    rng = np.random.default_rng(a + b)
    wide = lambda n: rng.integers(-(1 << 62), 1 << 62, n)
    rk = rng.permutation(np.concatenate([wide(5000), np.full(a, 11), np.full(a + 1, 12)]))
    sk = rng.permutation(np.concatenate([rng.choice(rk, 3000), np.full(b, 11), np.full(b // 2, 12)]))
    rr, sr = rng.permutation(rk.size).astype(np.int32), rng.permutation(sk.size).astype(np.int32)
    xr, xs, cnt = oracle.join_pairs(rk, rr, sk, sr)
    pr, ps = tj.join(dev(rk), dev(rr), dev(sk), dev(sr), capacity=cnt)
    assert np.array_equal(pr.cpu().numpy(), xr) and np.array_equal(ps.cpu().numpy(), xs)
