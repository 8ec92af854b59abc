"""Small requests that share calls use every slot: the calls of a burst overlap."""
import time

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("slots", [2, 4])
def test_calls_of_a_burst_overlap(slots):
    import paper_2602_21237_amd as tj
    tj.load()
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    reqs = []
    for i in range(320):
        k = torch.randint(0, 1 << 30, (200 + 90 * i,), device="cuda", generator=g)
        if i % 2:
            k = k.to(torch.int32)
        r = torch.arange(k.numel(), dtype=torch.int32, device="cuda")
        reqs.append((k, r, torch.empty_like(k), torch.empty_like(r)))
    overlap = []
    with tj.tj.Server(2 << 30, slots=slots) as srv:
        for _ in range(6):
            t0 = time.perf_counter()
            tickets = [srv.sort(*q) for q in reqs]
            res = [srv.wait(t) for t in tickets]
            span = (time.perf_counter() - t0) * 1e3
            assert all(r["status"] == 0 for r in res) and max(r["fused"] for r in res) > 1
            overlap.append(sum(r["run_ms"] / r["fused"] for r in res) / span)  # time of all calls, to the burst's
    for (k, r, ko, ro), q in zip(reqs, res):
        assert torch.equal(ko, torch.sort(k, stable=True).values)
    # calls one after the other give at most 1 on one slot
    assert max(overlap[1:]) > 0.7 * slots, overlap
