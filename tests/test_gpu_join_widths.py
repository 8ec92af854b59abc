"""Joins whose leaves' keys are narrowed in every second bucket: one launch takes
leaves of either width. Against the oracle, with the sorted way too."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.mark.parametrize("force", [False, True])
@pytest.mark.parametrize("keys,rows_a_key,n_s", [(1_000_000, 1, 4_000_000), (100_000, 60, 300_000)])
def test_alternating_widths(keys, rows_a_key, n_s, force):
    import paper_2602_21237_amd as tj
    tj.load()
    rng = np.random.default_rng(keys)
    high = rng.integers(0, 512, keys, dtype=np.int64) - 256
    low = np.where(high % 2 == 0, rng.integers(0, 1 << 55, keys), rng.integers(0, 1 << 20, keys))
    rk = rng.permutation(np.repeat(high * (1 << 55) + low, rows_a_key))
    sk = rk[rng.integers(0, rk.size, n_s)]
    rr, sr = rng.permutation(rk.size).astype(np.int32), rng.permutation(sk.size).astype(np.int32)
    xr, xs, cnt = oracle.join_pairs(rk, rr, sk, sr)
    tj.tj.debug_set_flags(tj.tj.TJ_DEBUG_FORCE_REORDER if force else 0)
    try:
        tj.timing(True)
        pr, ps = tj.join(dev(rk), dev(rr), dev(sk), dev(sr), capacity=cnt + 1)
        launches = tj.timing_read()["leaf_join_mat"]["launches"]
    finally:
        tj.timing(False)
        tj.tj.debug_set_flags(0)
    assert np.array_equal(pr.cpu().numpy(), xr) and np.array_equal(ps.cpu().numpy(), xs)
    assert launches < 20, launches
