"""The LDS block of the sort, in its shapes for few leaves and for many (over
256): even keys, bins of as many rows as the counting way takes and one more, and
the crowded leaves of the digit passes: many rows a key, few and many rows that
share their top 32 bits and differ below. Values and order are exact."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FEW, MANY = 9_001, 2_300_001


@pytest.fixture(scope="module")
def tj():
    import paper_2602_21237_amd as p
    p.load()
    return p


def keys_of(kind, n, rng):
    wide = rng.integers(-(1 << 62), 1 << 62, n)
    if kind == "even":
        return wide
    if kind == "even32":
        return rng.integers(-(1 << 31), 1 << 31, n).astype(np.int32)
    if kind in ("bin48", "bin49"):  # one key of 48 (49) rows in every stretch of some thousands
        m = int(kind[3:])
        k = wide.copy()
        for i in range(0, n - m, 5000):
            k[i:i + m] = k[i]
        return rng.permutation(k)
    if kind == "rows64":  # 64 rows a key
        return rng.choice(wide[: max(n // 64, 1)], n)
    if kind == "rows64_32":
        return rng.choice(wide[: max(n // 64, 1)], n).astype(np.int32)
    # crowded keys whose rows differ in low bits: all of them, or a few
    head = rng.choice(wide[: max(n // 64, 1)], n) & ~np.int64((1 << 12) - 1)
    low = rng.integers(0, 1 << 12, n)
    if kind == "few_ties":
        low[rng.random(n) > 2e-3] = 0
    return head + low


@pytest.mark.parametrize("n", [FEW, MANY])
@pytest.mark.parametrize("kind", ["even", "even32", "bin48", "bin49", "rows64", "rows64_32", "ties", "few_ties"])
def test_leaf_sort(tj, kind, n):
    rng = np.random.default_rng(n)
    k = keys_of(kind, n, rng)
    r = rng.integers(-(1 << 31), 1 << 31, n).astype(np.int32)
    ko, ro, st = tj.sort(torch.from_numpy(k).cuda(), torch.from_numpy(r).cuda(), stats=True)
    o = np.argsort(k, kind="stable")
    assert np.array_equal(ko.cpu().numpy(), k[o]) and np.array_equal(ro.cpu().numpy(), r[o])
    assert (st["leaves"] > 256) == (n == MANY), st
