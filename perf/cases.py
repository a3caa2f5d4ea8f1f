"""Workloads of the join and group-by library, through its Python entry points.

Every case is one call (or one launch of a plan) on device-resident columns, as a
query engine makes it: small lookups where launches count, the join and group-by
sizes of the paper's evaluation, odd row counts between them, 4- and 8-byte keys and
payloads, partial matches, skew, many-to-many keys, and batches held in a plan.

`listed()` names the fixed cases, `draw(rng)` gives one more of the same ranges,
`prepare` makes the inputs on the GPU (and a plan where a program would keep one),
`run` is one pass, `work` the bytes the pass cannot do without, and `exact` the same
result from plain torch where the row order of the result is specified.
"""
from __future__ import annotations

import random

import torch

import paper_2312_00720_amd as gj

DEV = "cuda"
SUM_ALL = "count+sum+min+max"  # COUNT, and SUM, MIN, MAX of every value column
MAX_ALL = "max"                # the paper's group-by aggregate: MAX of every value column


def _join(name, n_r, n_s, pay, *, key64=False, wide=0, match=1.0, alpha=0.0, keys=0):
    """keys > 0: a many-to-many join whose keys are drawn from that many values on both
    sides; else PK-FK. pay payload columns a side, the last `wide` of them 8 bytes."""
    c = {"kind": "join", "n_r": n_r, "n_s": n_s, "pay": pay, "key64": key64, "wide": wide, "match": match,
         "alpha": alpha, "keys": keys}
    return dict(c, name=name) if name else c


def _groupby(name, n, g, vals, *, aggs=SUM_ALL, algo="auto", ordered=False, key64=False, wide=0, alpha=0.0):
    c = {"kind": "groupby", "n": n, "g": g, "vals": vals, "aggs": aggs, "algo": algo, "ordered": ordered,
         "key64": key64, "wide": wide, "alpha": alpha}
    return dict(c, name=name) if name else c


def _partition(name, n, cols, bits, mode, *, key64=False):
    c = {"kind": "partition", "n": n, "cols": cols, "bits": bits, "mode": mode, "key64": key64}
    return dict(c, name=name) if name else c


def _plan(name, kind, instances, lo, hi, cols, shape):
    """A batch of `instances` joins or group-bys with round(2^U(lo, hi)) rows each
    (shape seeds the sizes: a plan is made for them)."""
    c = {"kind": kind, "instances": instances, "lo": lo, "hi": hi, "cols": cols, "shape": shape}
    return dict(c, name=name) if name else c


def listed():
    return [
        # a dimension lookup of a short query: latency and launches
        _join("join_small", 1000, 4000, 1),
        # the small join configuration (|R| = 2^16, |S| = 2^20, one payload a side)
        _join("join_c1", 1 << 16, 1 << 20, 1),
        # an ordinary join: 8-byte keys and one 8-byte payload a side, odd sizes, half the rows match, skewed FKs
        _join("join_key64_skew", 1_500_001, 12_000_007, 2, key64=True, wide=1, match=0.5, alpha=1.0),
        # the headline join (|R| = 2^27, |S| = 2^28, four payloads a side)
        _join("join_c2", 1 << 27, 1 << 28, 4),
        # many-to-many: four rows a side and key, four matches per row
        _join("join_m2n", 1 << 24, 1 << 24, 2, keys=1 << 22),
        # the partition primitive on its own (a shuffle or an exchange by hash)
        _partition("partition", (1 << 25) + 77, 2, 7, "hash"),
        # a small report, ordered by key
        _groupby("groupby_small", 10_007, 100, 2, ordered=True),
        # few groups over many rows, ordered by key (the automatic choice hashes)
        _groupby("groupby_few", 1 << 26, 1000, 2, ordered=True),
        # the paper's group-by size, N = 2^28 rows over 2^16 keys (the automatic choice partitions)
        _groupby("groupby_c3", 1 << 28, 1 << 16, 2),
        # ordered output over many skewed 8-byte keys and 8-byte values, the paper's MAX aggregate
        _groupby("groupby_sort64", (1 << 24) + 4099, 1 << 20, 2, aggs=MAX_ALL, algo="sort", key64=True, wide=1,
                 alpha=1.0),
        # many small joins and group-bys planned once and launched as one graph
        _plan("join_plan", "join_plan", 512, 8, 18, 2, 3),
        _plan("groupby_plan", "groupby_plan", 512, 8, 18, 2, 4),
    ]


def _size(rng, lo, hi):
    """An odd-ish size, uniform in its logarithm between 2^lo and 2^hi."""
    return int(round(2.0 ** rng.uniform(lo, hi)))


def draw(rng: random.Random):
    kind = rng.choice(["join", "join", "join", "m2n", "partition", "groupby", "groupby", "few", "sort", "join_plan",
                       "groupby_plan"])
    if kind == "join":
        n_r = _size(rng, 8, 25)
        n_s = min(1 << 27, int(n_r * rng.uniform(1, 16)))
        pay = rng.randint(1, 4)
        return _join(None, n_r, n_s, pay, key64=rng.random() < 0.3, wide=rng.randint(0, 1), match=rng.choice([1.0, 1.0, 0.5]),
                     alpha=rng.choice([0.0, 0.0, 0.5, 1.0]))
    if kind == "m2n":
        n = _size(rng, 10, 24)
        return _join(None, n, int(n * rng.uniform(1, 2)), rng.randint(1, 2), keys=max(1, n // rng.randint(2, 4)))
    if kind == "partition":
        return _partition(None, _size(rng, 10, 27), rng.randint(0, 4), rng.randint(2, 12), rng.choice(["bits", "hash"]),
                          key64=rng.random() < 0.3)
    if kind in ("groupby", "sort"):
        n = _size(rng, 13, 27 if kind == "groupby" else 25)
        g = max(2, min(n // 4, _size(rng, 8, 23)))
        return _groupby(None, n, g, rng.randint(1, 3), aggs=rng.choice([SUM_ALL, MAX_ALL]),
                        algo="partition" if kind == "groupby" else "sort", key64=rng.random() < 0.3,
                        wide=rng.randint(0, 1), alpha=rng.choice([0.0, 0.0, 1.0]))
    if kind == "few":
        return _groupby(None, _size(rng, 13, 27), _size(rng, 2, 11), rng.randint(1, 3), ordered=True,
                        aggs=rng.choice([SUM_ALL, MAX_ALL]), key64=rng.random() < 0.3)
    return _plan(None, kind, _size(rng, 5, 10), 8, rng.randint(12, 18), rng.randint(1, 2), rng.randrange(1 << 20))


# ---- inputs ------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 2654435761 % (1 << 62))
    return g


def _wide_keys(k):
    """A bijection of small key values onto all 64 bits (multiply by odd constants, xor shifts)."""
    z = k.to(torch.int64) * -7046029254386353131
    z = (z ^ ((z >> 32) & 0xFFFFFFFF)) * -4658895280553007687
    return z ^ ((z >> 29) & ((1 << 35) - 1))


def _ranks(g, count, n, alpha):
    """`count` values in 0..n-1, uniform or with P(i) ~ (i + 1)^-alpha."""
    if alpha == 0.0:
        return torch.randint(0, n, (count,), generator=g, device=DEV, dtype=torch.int64)
    cdf = torch.cumsum(torch.arange(1, n + 1, device=DEV, dtype=torch.float64).pow_(-alpha), 0)
    u = torch.rand(count, generator=g, device=DEV, dtype=torch.float64) * cdf[-1]
    return torch.searchsorted(cdf, u, right=True).clamp_(max=n - 1)


def _columns(g, n, count, wide, lo=-(2 ** 31), hi=2 ** 31 - 1):
    out = []
    for j in range(count):
        dt = torch.int64 if j >= count - wide else torch.int32
        out.append(torch.randint(lo, hi, (n,), generator=g, device=DEV, dtype=dt))
    return out


def _aggs(case):
    if case["aggs"] == MAX_ALL:
        return [(c, "max") for c in range(case["vals"])]
    return [(0, "count")] + [(c, op) for c in range(case["vals"]) for op in ("sum", "min", "max")]


def _plan_sizes(case):
    rng = random.Random(case["shape"])
    first = [_size(rng, case["lo"], case["hi"]) for _ in range(case["instances"])]
    second = [int(n * rng.uniform(1, 4)) for n in first]
    return first, second


def _offsets(sizes):
    off = [0]
    for n in sizes:
        off.append(off[-1] + n)
    return off


def _instances(sizes):
    s = torch.tensor(sizes, device=DEV)
    return torch.repeat_interleave(torch.arange(len(sizes), device=DEV), s)


def _shuffled(g, sizes):
    """A random permutation of 0..n-1 for every instance of n rows, back to back."""
    inst = _instances(sizes)
    rnd = torch.randint(0, 1 << 40, (inst.numel(),), generator=g, device=DEV)
    return torch.argsort((inst << 40) | rnd) - torch.tensor(_offsets(sizes)[:-1], device=DEV)[inst]


def _matches(case):
    """S rows of a PK-FK join that find their key in R."""
    return round(case["match"] * case["n_s"])


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    if kind == "join":
        n_r, n_s, keys = case["n_r"], case["n_s"], case["keys"]
        r = torch.randperm(n_r, generator=g, device=DEV)
        if keys:  # every value occurs equally often (up to one) on each side, in a random order
            r, s = r % keys, torch.randperm(n_s, generator=g, device=DEV) % keys
        else:
            s = _ranks(g, n_s, n_r, case["alpha"])
            if case["match"] < 1.0:
                miss = torch.randperm(n_s, generator=g, device=DEV)[_matches(case):]
                s[miss] = torch.randint(n_r, 2 ** 31, (miss.numel(),), generator=g, device=DEV)
        r, s = (_wide_keys(r), _wide_keys(s)) if case["key64"] else (r.to(torch.int32), s.to(torch.int32))
        wide = min(case["wide"], case["pay"])
        return {"case": case, "cols": (r, _columns(g, n_r, case["pay"], wide), s, _columns(g, n_s, case["pay"], wide))}
    if kind == "groupby":
        k = _ranks(g, case["n"], case["g"], case["alpha"])
        k[torch.randperm(case["n"], generator=g, device=DEV)[:case["g"]]] = torch.arange(case["g"], device=DEV)  # no empty group
        k = _wide_keys(k) if case["key64"] else k.to(torch.int32)
        vals = _columns(g, case["n"], case["vals"], min(case["wide"], case["vals"]), -(2 ** 20), 2 ** 20 + 1)
        return {"case": case, "cols": (k, vals, _aggs(case))}
    if kind == "partition":
        k = torch.randint(0, 2 ** 31, (case["n"],), generator=g, device=DEV)
        k = _wide_keys(k) if case["key64"] else k.to(torch.int32)
        return {"case": case, "cols": (k, _columns(g, case["n"], case["cols"], 0))}
    first, second = _plan_sizes(case)
    if kind == "join_plan":
        r = _shuffled(g, first)
        size = torch.tensor(first, device=DEV)[_instances(second)]
        s = torch.minimum((torch.rand(size.numel(), generator=g, device=DEV, dtype=torch.float64) * size).long(), size - 1)
        plan = gj.JoinPlan(r.to(torch.int32), _columns(g, r.numel(), case["cols"], 0), _offsets(first),
                           s.to(torch.int32), _columns(g, s.numel(), case["cols"], 0), _offsets(second))
    else:
        card = torch.tensor([max(4, n // 16) for n in first], device=DEV)[_instances(first)]
        k = _shuffled(g, first) % card
        vals = _columns(g, k.numel(), case["cols"], 0, -(2 ** 20), 2 ** 20 + 1)
        plan = gj.GroupByPlan(k.to(torch.int32), vals, _offsets(first), _aggs(dict(aggs=SUM_ALL, vals=case["cols"])))
    plan.capture()
    return {"case": case, "plan": plan}


# ---- one pass ------------------------------------------------------------------------

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "join":
        key, r, s = gj.join(*state["cols"])
        return [key, *r, *s]
    if kind == "groupby":
        key, aggs = gj.groupby(*state["cols"], algo=case["algo"])
        if case["ordered"]:  # ... ORDER BY key: the hash group-by's own order is unspecified
            key, order = torch.sort(key)
            aggs = [a[order] for a in aggs]
        return [key, *aggs]
    if kind == "partition":
        key, cols, _, off = gj.partition(*state["cols"], bits=case["bits"], mode=case["mode"])
        return [key, *cols, off]
    plan = state["plan"]
    plan.launch()
    out = plan.result()
    if kind == "join_plan":
        return [out[0], *out[1], *out[2], out[3][-1]]
    return [out[0], *out[1], out[2][-1]]


# ---- what a pass cannot do without ----------------------------------------------------

def _agg_bytes(case, kb):
    b = kb
    wide = min(case["wide"], case["vals"])
    for c, op in _aggs(case):
        b += 8 if op in ("sum", "count") or c >= case["vals"] - wide else 4
    return b


def work(case):
    """Every input column read once and every output column written once."""
    kind = case["kind"]
    if kind == "join":
        row = (8 if case["key64"] else 4) + 4 * case["pay"] + 4 * min(case["wide"], case["pay"])
        pay = row - (8 if case["key64"] else 4)
        t = case["n_r"] * case["n_s"] / case["keys"] if case["keys"] else _matches(case)
        return {"bytes": (case["n_r"] + case["n_s"]) * row + t * (row + pay), "flops": 0}
    if kind == "groupby":
        kb = 8 if case["key64"] else 4
        row = kb + 4 * case["vals"] + 4 * min(case["wide"], case["vals"])
        return {"bytes": case["n"] * row + min(case["g"], case["n"]) * _agg_bytes(case, kb), "flops": 0}
    if kind == "partition":
        row = (8 if case["key64"] else 4) + 4 * case["cols"]
        return {"bytes": 2 * case["n"] * row + 4 * ((1 << case["bits"]) + 1), "flops": 0}
    first, second = _plan_sizes(case)
    row = 4 + 4 * case["cols"]
    if kind == "join_plan":
        return {"bytes": (sum(first) + sum(second)) * row + sum(second) * (row + 4 * case["cols"]), "flops": 0}
    g = sum(max(4, n // 16) for n in first)
    return {"bytes": sum(first) * row + g * (12 + 16 * case["cols"]), "flops": 0}


# ---- the same result from plain torch ---------------------------------------------------

def _fmix32(x):
    """MurmurHash3's 32-bit finalizer on int64 tensors holding 32-bit values."""
    m = 0xFFFFFFFF
    x = x ^ (x >> 16)
    x = (x * 0x85EBCA6B) & m
    x = x ^ (x >> 13)
    x = (x * 0xC2B2AE35) & m
    return x ^ (x >> 16)


def exact(case, seed):
    """Joins, plans and the partition group-by leave their row order unspecified: None."""
    kind = case["kind"]
    if kind == "partition":
        key, cols = prepare(case, seed)["cols"]
        u = key.to(torch.int64)
        if case["mode"] == "hash":
            u = u & 0xFFFFFFFF if not case["key64"] else (u ^ (u >> 32)) & 0xFFFFFFFF
            u = _fmix32(u)
        digit = u & ((1 << case["bits"]) - 1)
        order = torch.sort(digit, stable=True).indices
        count = torch.bincount(digit, minlength=1 << case["bits"])
        off = torch.cat([count.new_zeros(1), torch.cumsum(count, 0)])
        return [key[order], *[c[order] for c in cols], off.to(torch.int32)]
    if kind == "groupby" and (case["ordered"] or case["algo"] == "sort"):
        key, vals, aggs = prepare(case, seed)["cols"]
        keys, inv = torch.unique(key, return_inverse=True)
        out = [keys]
        for c, op in aggs:
            v = vals[c].to(torch.int64)
            if op == "count":
                out.append(torch.bincount(inv, minlength=keys.numel()))
            elif op == "sum":
                out.append(torch.zeros(keys.numel(), dtype=torch.int64, device=DEV).index_add_(0, inv, v))
            else:
                z = torch.zeros(keys.numel(), dtype=torch.int64, device=DEV)
                z.scatter_reduce_(0, inv, v, "amin" if op == "min" else "amax", include_self=False)
                out.append(z.to(vals[c].dtype))
        return out
    return None
