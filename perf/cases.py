"""The work that programs have this library do, as cases that can be timed.

Keys and row ids are made on the GPU from a seed. The relations follow the
shapes that the benchmark and the tests use: uniform int32 keys over 20 bits
(R and S of 10^5 rows), foreign-key pairs (unique 40-bit R keys; 80% of S
takes an R key, uniformly or by Zipf(0.99) rank, 20% keys that R lacks),
64-bit uniform and lognormal(30, 2) sort keys, and queues of requests of
uneven sizes. Outputs are the sorted columns, the pair count, or the pairs in
canonical order. A case that returns pairs has as many for one seed as for
another.
"""
import math
import random
import weakref

import torch

import paper_2602_21237_amd as tj
from paper_2602_21237_amd.tj import Server

MASK40 = (1 << 40) - 1
MATCHED = 0.8          # share of S rows that take a key of R
HOT_MULT = 4           # copies in R of each of its hottest keys, where "hot" is not 0
DTYPE = {"i32": torch.int32, "i64": torch.int64}
KEY_BYTES = {"i32": 4, "i64": 8}


def listed():
    return [
        # the smallest call: a lookup result or a group of rows put in order
        dict(name="sort_1k_i32", op="sort", rows=1000, key="i32", dist="uniform32", budget=0, part="radix"),
        # the small workload of the benchmark, |R| = |S| = 10^5
        dict(name="sort_100k_i32", op="sort", rows=100_000, key="i32", dist="uniform20", budget=0, part="radix"),
        # the same relations joined by a caller who does not know the result's
        # size: a count, then the pairs
        dict(name="join_100k_i32", op="join", n_r=100_000, n_s=100_000, key="i32", dist="uniform20", theta=0.0,
             hot=0, budget=0, part="radix", known=False),
        # the paper-shaped workload, N = 10^6: a sort of skewed foreign keys
        dict(name="sort_1m_zipf", op="sort", rows=1_000_000, key="i64", dist="fk", theta=0.99, budget=0,
             part="radix"),
        # ... its join with enough memory
        dict(name="join_1m", op="join", n_r=1_000_000, n_s=1_000_000, key="i64", dist="fk", theta=0.0, hot=0,
             budget=0, part="radix", known=True),
        # ... and under the paper's work_mem of 1 MB
        dict(name="join_1m_1mib", op="join", n_r=1_000_000, n_s=1_000_000, key="i64", dist="fk", theta=0.0, hot=0,
             budget=1 << 20, part="radix", known=True),
        # a join over two key columns (an int32 and an int64), packed into one
        dict(name="join_two_columns_5m", op="join_multi", n_r=5_000_011, n_s=5_000_011),
        # a queue of sorts and joins of uneven sizes, all waiting at once
        dict(name="serve_24", op="serve", requests=24, lo=1000, hi=1_000_000, slots=8),
        # heavy-tailed keys, where the call picks its partitioner itself
        dict(name="sort_100m_lognormal_auto", op="sort", rows=100_000_007, key="i64", dist="lognormal", budget=0,
             part="auto"),
        # the size of a skewed join: hot keys repeated on both sides
        dict(name="count_zipf_2p28", op="count", n_r=1 << 26, n_s=1 << 28, key="i64", dist="fk", theta=0.99,
             hot=1 << 19, budget=0, part="radix"),
        # the benchmark's own step: the sort of 2^29 rows and the join of 2^27 with 2^29
        dict(name="sort_2p29", op="sort", rows=1 << 29, key="i64", dist="uniform64", budget=0, part="radix"),
        dict(name="join_2p27_2p29", op="join", n_r=1 << 27, n_s=1 << 29, key="i64", dist="fk", theta=0.0, hot=0,
             budget=0, part="radix", known=True),
    ]


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    kind = rng.choice(["sort", "sort", "sort", "join", "join", "join", "count", "budget", "join_multi", "serve"])
    key = rng.choice(["i32", "i64", "i64"])
    if kind == "sort":
        dist = rng.choice(["uniform32", "uniform20"] if key == "i32" else ["uniform64", "fk", "lognormal"])
        part = "auto" if dist == "lognormal" and rng.random() < 0.5 else "radix"
        return dict(op="sort", rows=_log_uniform(rng, 1000, 1 << 28), key=key, dist=dist,
                    theta=rng.choice([0.0, 0.8, 0.99]), budget=0, part=part)
    if kind in ("join", "count"):
        n_r = _log_uniform(rng, 1000, 1 << 26)
        n_s = _log_uniform(rng, 1000, 1 << 27)
        theta = rng.choice([0.0, 0.8, 0.99])
        if key == "i32":  # at most about half as many pairs as S rows
            n_r, n_s = min(n_r, 1 << 19), min(n_s, 1 << 20)
        return dict(op=kind, n_r=n_r, n_s=n_s, key=key, dist="uniform20" if key == "i32" else "fk", theta=theta,
                    hot=n_r // 128 if theta == 0.99 else 0, budget=0, part="radix", known=rng.random() < 0.7)
    if kind == "budget":
        budget = _log_uniform(rng, 1 << 20, 64 << 20)
        if rng.random() < 0.5:
            return dict(op="sort", rows=_log_uniform(rng, 100_000, 4_000_000), key="i64", dist="fk",
                        theta=rng.choice([0.0, 0.99]), budget=budget, part="radix")
        n = _log_uniform(rng, 100_000, 1_200_000)
        return dict(op="join", n_r=n, n_s=n, key="i64", dist="fk", theta=rng.choice([0.0, 0.99]), hot=0,
                    budget=budget, part="radix", known=True)
    if kind == "join_multi":
        return dict(op="join_multi", n_r=_log_uniform(rng, 10_000, 1 << 24), n_s=_log_uniform(rng, 10_000, 1 << 24))
    return dict(op="serve", requests=rng.randint(8, 30), lo=1000, hi=_log_uniform(rng, 10_000, 2_000_000),
                slots=rng.choice([4, 8]))


# --------------------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _scramble40(x, salt):
    """A bijection of [0, 2^40), another one for each salt."""
    a = (salt * 0x9E3779B97F4A7 + 0x2545F4914F6CDD1D) & MASK40 | 1
    b = (salt * 0x2127599BF4325 + 0x5851F42D4C957F2D) & MASK40 | 1
    x = (x * a + salt) & MASK40
    x = x ^ (x >> 19)
    x = (x * b) & MASK40
    return x ^ (x >> 21)


def _zipf_ranks(n, d, theta, hot, g):
    """n ranks in [0, d), rank r with a density of about (r + 1)^-theta. With `hot`, rows are told off beforehand
    to ranks below it or not, by the share that these have."""
    if theta == 0.0:
        return torch.randint(0, d, (n,), device="cuda", generator=g)
    u = torch.rand(n, dtype=torch.float64, device="cuda", generator=g)
    if hot:
        share = _zipf_share(d, theta, hot)
        u = torch.where(_is_hot(n, share), u * share, u * (1.0 - share) + share)
    e = 1.0 - theta
    u.mul_(float(d + 1) ** e - 1.0).add_(1.0).pow_(1.0 / e)
    ranks = u.to(torch.int64).sub_(1).clamp_(0, d - 1)
    if hot:  # rounding at the border between the two
        h = _is_hot(n, share)
        ranks = torch.where(h, ranks.clamp(max=hot - 1), ranks.clamp(min=hot))
    return ranks


def _is_hot(n, share):
    return torch.arange(n, device="cuda") % 1009 < round(1009 * share)


def _zipf_share(d, theta, hot):
    """The share of the ranks of _zipf_ranks that lie below `hot`."""
    if theta == 0.0:
        return hot / d
    e = 1.0 - theta
    return (float(hot + 1) ** e - 1.0) / (float(d + 1) ** e - 1.0)


def _fk_pair(n_r, n_s, theta, hot, salt, g, fixed=True):
    """R's keys (its `hot` first ranks HOT_MULT times each) and S's keys; `fixed`: with the same number of pairs
    for every seed."""
    d = n_r - hot * (HOT_MULT - 1)
    at = torch.arange(n_r, device="cuda")
    if hot:
        at = torch.where(at < d, at, (at - d) % hot)
        # copies of a key lie apart, as rows of a table do
        at = at[torch.randperm(n_r, device="cuda", generator=g)]
    r = _scramble40(at, salt)
    return r, _fk_keys(n_s, d, theta, hot, salt, g, fixed)


def _fk_keys(n_s, d, theta, hot, salt, g, fixed):
    at = torch.arange(n_s, device="cuda")
    miss = at % 5 == 4 if fixed else torch.rand(n_s, device="cuda", generator=g) >= MATCHED
    return _scramble40(torch.where(miss, at + d, _zipf_ranks(n_s, d, theta, hot if fixed else 0, g)), salt)


def _sort_keys(case, seed, g):
    n, dist = case["rows"], case["dist"]
    if dist == "uniform32":
        return torch.randint(-(1 << 31), 1 << 31, (n,), device="cuda", generator=g).to(torch.int32)
    if dist == "uniform20":
        return torch.randint(0, 1 << 20, (n,), device="cuda", generator=g).to(DTYPE[case["key"]])
    if dist == "uniform64":
        hi = torch.randint(-(1 << 31), 1 << 31, (n,), device="cuda", generator=g)
        return (hi << 32) + torch.randint(0, 1 << 32, (n,), device="cuda", generator=g)
    if dist == "lognormal":
        z = torch.randn(n, dtype=torch.float64, device="cuda", generator=g)
        return z.mul_(2.0).add_(30.0).exp_().to(torch.int64)
    return _fk_keys(n, n, case["theta"], 0, seed, g, True)  # the S side of a foreign-key pair


def _rids(n):
    return torch.arange(n, dtype=torch.int32, device="cuda")


def _relations(case, seed):
    g = _gen(seed)
    if case["dist"] == "uniform20":
        # uniform keys, for pairs those of one draw relabelled and shuffled by the seed
        fixed, sides = g if case["op"] == "count" else _gen(20), []
        for n in (case["n_r"], case["n_s"]):
            k = torch.randint(0, 1 << 20, (n,), device="cuda", generator=fixed)
            k = (k * (2 * seed * 0x9E375 + 0x3C6EF) + seed) & 0xFFFFF  # an odd factor: a bijection
            sides.append(k[torch.randperm(n, device="cuda", generator=g)].to(DTYPE[case["key"]]))
        return sides
    return _fk_pair(case["n_r"], case["n_s"], case["theta"], case["hot"], seed, g, case["op"] != "count")


def _columns(case, seed):
    """Two key columns a side: a foreign key's 40 bits as (int32, int64)."""
    r, s = _fk_pair(case["n_r"], case["n_s"], 0.0, 0, seed, _gen(seed))
    return [[(k >> 20).to(torch.int32), (k & 0xFFFFF) - (1 << 19)] for k in (r, s)]


def _requests(case, seed):
    """The queue's requests: (operation, keys...), sizes log-uniform in [lo, hi]."""
    g = _gen(seed)
    sizes = random.Random(case["requests"])
    out = []
    for i in range(case["requests"]):
        n_r, n_s = (_log_uniform(sizes, case["lo"], case["hi"]) for _ in range(2))
        r, s = _fk_pair(n_r, n_s, 0.8 if i % 2 else 0.0, 0, seed * 64 + i, g)
        out.append(("sort", s) if (i // 2) % 2 else ("join", r, s))
    return out


# --------------------------------------------------------------------------- state and pass

class _Queue:
    """A running server and the requests that wait for it."""

    def __init__(self, case, seed):
        self.server = Server(2 << 30, slots=case["slots"])
        weakref.finalize(self, self.server.close)
        self.items = []
        for op, *keys in _requests(case, seed):
            rids = [_rids(k.numel()) for k in keys]
            if op == "sort":
                outs = (torch.empty_like(keys[0]), torch.empty_like(rids[0]))
            else:  # a row of S matches one row of R at most
                outs = tuple(torch.empty(keys[1].numel(), dtype=torch.int32, device="cuda") for _ in range(2))
            self.items.append((op, keys, rids, outs))


def prepare(case, seed):
    op = case["op"]
    if op == "serve":
        return _Queue(case, seed)
    s = {"op": op, "part": case.get("part", "radix")}
    if op == "sort":
        s["keys"] = _sort_keys(case, seed, _gen(seed))
        s["rids"] = _rids(case["rows"])
        if case["rows"] >= 1 << 20 or case["budget"]:  # programs with large columns keep the outputs and workspace
            need = case["budget"] or tj.workspace_query(tj.TJ_OP_SORT, KEY_BYTES[case["key"]], case["rows"])[1]
            s["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
            s["out"] = (torch.empty_like(s["keys"]), torch.empty_like(s["rids"]))
        return s
    if op == "join_multi":
        s["r"], s["s"] = _columns(case, seed)
        s["rr"], s["sr"] = _rids(case["n_r"]), _rids(case["n_s"])
        return s
    s["r"], s["s"] = _relations(case, seed)
    if op == "join":
        s["rr"], s["sr"] = _rids(case["n_r"]), _rids(case["n_s"])
        if case["known"]:
            cap = case["n_s"] * (HOT_MULT if case["hot"] else 1)
            s["out"] = tuple(torch.empty(cap, dtype=torch.int32, device="cuda") for _ in range(2))
    if op == "count" or case["known"]:
        code = tj.TJ_OP_JOIN_COUNT if op == "count" else tj.TJ_OP_JOIN_MATERIALIZE
        need = case["budget"] or tj.workspace_query(code, KEY_BYTES[case["key"]], case["n_r"], case["n_s"])[1]
        s["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    return s


def run(state):
    if isinstance(state, _Queue):
        tickets = []
        for op, keys, rids, outs in state.items:
            if op == "sort":
                tickets.append(state.server.sort(keys[0], rids[0], outs[0], outs[1]))
            else:
                tickets.append(state.server.join(keys[0], rids[0], keys[1], rids[1], outs[0].numel(), outs[0], outs[1]))
        done = [state.server.wait(t) for t in tickets]
        return [(d["keys"], d["rids"]) if "keys" in d else (d["out_r"], d["out_s"]) for d in done]
    op, ws, out = state["op"], state.get("ws"), state.get("out", (None, None))
    if op == "sort":
        return tj.sort(state["keys"], state["rids"], out[0], out[1], workspace=ws, partitioner=state["part"])
    if op == "count":
        return tj.join_count(state["r"], state["s"], workspace=ws, partitioner=state["part"])
    if op == "join_multi":
        return tj.join_multi(state["r"], state["rr"], state["s"], state["sr"])
    return tj.join(state["r"], state["rr"], state["s"], state["sr"], out_r=out[0], out_s=out[1], workspace=ws,
                   partitioner=state["part"])


# --------------------------------------------------------------------------- floors and values

def _pairs(case):
    """Expected pairs of a join."""
    if case.get("dist") == "uniform20":
        return case["n_r"] * case["n_s"] / 2.0 ** 20
    hot = case.get("hot", 0)
    share = _zipf_share(case["n_r"] - hot * (HOT_MULT - 1), case["theta"], hot) if hot else 0.0
    return MATCHED * case["n_s"] * (1.0 + (HOT_MULT - 1) * share)


def work(case):
    """Each key and row id read once and each output written once; no arithmetic to speak of."""
    op = case["op"]
    if op == "serve":  # half sorts of S, half joins; sizes log-uniform
        mean = (case["hi"] - case["lo"]) / math.log(case["hi"] / case["lo"])
        return {"bytes": case["requests"] * mean * (0.5 * 24 + 0.5 * (24 + 8 * MATCHED)), "flops": 0.0}
    if op == "sort":
        return {"bytes": 2.0 * case["rows"] * (KEY_BYTES[case["key"]] + 4), "flops": 0.0}
    rows = case["n_r"] + case["n_s"]
    if op == "join_multi":
        return {"bytes": rows * 16.0 + 8.0 * MATCHED * case["n_s"], "flops": 0.0}
    if op == "count":
        return {"bytes": float(rows * KEY_BYTES[case["key"]]), "flops": 0.0}
    return {"bytes": rows * (KEY_BYTES[case["key"]] + 4.0) + 8.0 * _pairs(case), "flops": 0.0}


def _exact_sort(keys):
    k, at = torch.sort(keys, stable=True)
    return k, at.to(torch.int32)


def _exact_matches(r, s):
    """R and S in stable key order, and for each R row in that order its first match in S's order and their number."""
    rk, ri = torch.sort(r, stable=True)
    sk, si = torch.sort(s, stable=True)
    lo = torch.searchsorted(sk, rk)
    n = torch.searchsorted(sk, rk, right=True) - lo
    return ri, si, lo, n


def _exact_join(r, s):
    ri, si, lo, n = _exact_matches(r, s)
    # pairs come by key, then R row, then S row; R's stable order is that order
    first = torch.cumsum(n, 0) - n
    i = torch.repeat_interleave(torch.arange(n.numel(), device=n.device), n)
    j = torch.arange(i.numel(), device=n.device) - first[i] + lo[i]
    return ri[i].to(torch.int32), si[j].to(torch.int32)


def exact(case, seed):
    op = case["op"]
    if op == "serve":
        return [_exact_sort(k[0]) if o == "sort" else _exact_join(*k) for o, *k in _requests(case, seed)]
    if op == "sort":
        return _exact_sort(_sort_keys(case, seed, _gen(seed)))
    if op == "join_multi":
        r, s = ([(c[0].to(torch.int64) << 20) + c[1]] for c in _columns(case, seed))
        return _exact_join(r[0], s[0])
    r, s = _relations(case, seed)
    if op == "count":
        return int(_exact_matches(r, s)[3].sum())
    return _exact_join(r, s)
