"""Joins of one block whose table crowds one bin: the R rows of many pairs go round the
block's waves. Against the oracle, with pairs on both sides of the 16 that a lane writes."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.mark.parametrize("dtype", [np.int32, np.int64])
@pytest.mark.parametrize("r_of,s_of", [
    ([490], [5089]),              # one key
    ([300, 1, 200], [15, 16, 17]),
    ([64, 65, 600, 1], [1, 900, 16, 500]),
    ([400] * 3, [8] * 3),          # lanes only
    ([900, 0, 17], [0, 50, 90]),
    ([4096], [4096]),
])
def test_join(r_of, s_of, dtype):
    import paper_2602_21237_amd as tj
    tj.load()
    g = np.random.default_rng(len(r_of))
    rk = g.permutation(np.repeat(np.arange(len(r_of)) * 3 - 2, r_of)).astype(dtype)
    sk = g.permutation(np.repeat(np.arange(len(s_of)) * 3 - 2, s_of)).astype(dtype)
    rr = g.permutation(rk.size).astype(np.int32)
    sr = g.permutation(sk.size).astype(np.int32)
    for swap in (False, True):
        if swap:
            rk, rr, sk, sr = sk, sr, rk, rr
        er, es, cnt = oracle.join_pairs(rk, rr, sk, sr)
        assert tj.join_count(dev(rk), dev(sk)) == cnt
        pr, ps = tj.join(dev(rk), dev(rr), dev(sk), dev(sr), capacity=cnt)
        assert np.array_equal(pr.cpu().numpy(), er) and np.array_equal(ps.cpu().numpy(), es)
        if cnt > 100:  # a capacity that ends inside a row's pairs
            out = torch.full((2, cnt), -7, dtype=torch.int32, device="cuda")
            with pytest.raises(tj.TjError):
                tj.join(dev(rk), dev(rr), dev(sk), dev(sr), capacity=cnt - 37, out_r=out[0], out_s=out[1])
            assert bool((out[:, cnt - 37:] == -7).all())
