"""Unlimited plans whose leaf table is smaller than the level that fills it: the
leaves batched on the device do not fit, and the level goes back to the host,
which plans it from the child records. tj_sort_static reaches this close to
the largest inputs of its unlimited plan (the scratch then leaves room for the
smallest tables only), tj_sort with a workspace just above its data buffers.
"""
import numpy as np
import pytest

import oracle
import tjgen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tj():
    import paper_2602_21237_amd as p
    p.load()
    return p


def _columns(n, dtype, seed):
    rng = np.random.default_rng(seed)
    info = np.iinfo(dtype)
    k = rng.integers(info.min, info.max, n, dtype=dtype, endpoint=True)
    return k, tjgen.perm_i32(n, seed)


@pytest.mark.parametrize("dtype,n", [(np.int64, 22_190_000), (np.int64, 22_300_000), (np.int64, 22_346_560),
                                     (np.int32, 33_300_000), (np.int32, 33_519_872)])
def test_static_sort_near_its_largest_plan(tj, dtype, n):
    print("tj_sort_static %s n=%d" % (np.dtype(dtype).name, n), flush=True)
    k, r = _columns(n, dtype, n % 97)
    dk, dr = torch.from_numpy(k).cuda(), torch.from_numpy(r).cuda()
    ek, er = tj.sort(dk, dr)
    # (earlier calls leave other records where the planner reads its own)
    small = torch.arange(100_000, 0, -1, dtype=dk.dtype, device="cuda")
    ids = torch.arange(100_000, dtype=torch.int32, device="cuda")
    tj.sort_static(small, ids, torch.empty_like(small), torch.empty_like(ids))
    ko, ro = torch.full_like(dk, 0x5A), torch.full_like(dr, 0x5A)
    st = tj.sort_static(dk, dr, ko, ro, stats=True)
    assert torch.equal(ko, ek) and torch.equal(ro, er)
    assert st["key_ranges"] == 1 and st["windows"] == 0 and st["leaves"] > 2048, st


@pytest.mark.parametrize("dtype,room", [(np.int64, 300 << 10), (np.int64, 600 << 10), (np.int32, 300 << 10)])
def test_sort_with_the_smallest_tables(tj, dtype, room):
    n = 9_000_000
    k, r = _columns(n, dtype, 3)
    dk, dr = torch.from_numpy(k).cuda(), torch.from_numpy(r).cuda()
    data = -(-n * dk.element_size() // 256) * 256 + -(-n * 4 // 256) * 256
    ko, ro, st = tj.sort(dk, dr, workspace_bytes=data + room, stats=True)
    assert st["key_ranges"] == 1 and st["windows"] == 0 and st["leaves"] > 1024, st
    ek, er = oracle.sort(k, r)
    assert np.array_equal(ko.cpu().numpy(), ek) and np.array_equal(ro.cpu().numpy(), er)
