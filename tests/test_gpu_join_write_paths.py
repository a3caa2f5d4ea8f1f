"""GPU parity of joins with few S rows of several matches, element by element: waves that
write in output order beside waves that do not, in one work unit and over the units
of a call, with R payloads in LDS or not; and the same keys through a plan."""
import numpy as np
import pytest

import datagen
import oracle

pytestmark = pytest.mark.gpu


def _data(n_r, n_s, extra, hit, kb, c_r, c_s, seed):
    """n_r distinct R keys, `extra` of them twice; `hit` S rows find one of those."""
    g = datagen.rng(seed)
    dt = np.int32 if kb == 4 else np.int64
    odd = 1 if kb == 4 else 0x5DEECE66D
    keys = g.permutation(2 * n_r)[:n_r].astype(np.int64)
    rk = g.permutation(np.concatenate([keys, keys[:extra]])) * odd
    sk = np.concatenate([g.choice(keys[:max(extra, 1)], size=hit), g.choice(keys[max(extra, 1):], size=n_s - hit)])
    sk = sk[np.argsort(np.concatenate([np.arange(hit) * 37 % n_s, g.integers(0, n_s, size=n_s - hit)]), kind="stable")] * odd
    cols = lambda n, c: [g.integers(-2**62, 2**62, size=n, dtype=np.int64) if j % 3 == 2
                         else g.integers(-2**31, 2**31, size=n, dtype=np.int64).astype(np.int32) for j in range(c)]
    return {"r_key": rk.astype(dt), "r_pay": cols(len(rk), c_r), "s_key": sk.astype(dt), "s_pay": cols(n_s, c_s)}


CASES = [
    # distinct R keys, S rows, keys twice, S rows that hit them, key bytes, R / S payloads, lds_budget, radix_bits
    (6000, 40000, 0, 0, 4, 2, 2, 4096, 1),
    (6000, 40000, 1, 1, 4, 2, 2, 4096, 1),      # one wave of one unit
    (6000, 40000, 3, 60, 4, 2, 2, 4096, 1),
    (6000, 40000, 600, 5000, 4, 2, 2, 4096, 1),
    (6000, 40000, 600, 5000, 4, 1, 1, 4096, 1),  # too few columns to write in order
    (6000, 40000, 600, 5000, 8, 3, 1, 4096, 1),
    (6000, 40000, 2, 30, 8, 1, 5, 4096, 1),
    (6000, 9000, 2, 7, 4, 4, 4, 4096, 1),        # units of four waves
    (12000, 70000, 2, 40, 8, 3, 3, 8192, 1),
    (28000, 150000, 4, 50, 4, 4, 2, 16384, 1),
]


@pytest.mark.parametrize("mat", ["gftr", "gfur"])
@pytest.mark.parametrize("case", CASES)
def test_mixed_waves(case, mat):
    import paper_2312_00720_amd as gj
    from gpu_util import dev, host, say
    n_r, n_s, extra, hit, kb, c_r, c_s, budget, bits = case
    say(f"join write paths {case} {mat}")
    d = _data(n_r, n_s, extra, hit, kb, c_r, c_s, seed=9000 + extra + kb)
    k, r, s = gj.join(dev(d["r_key"]), [dev(x) for x in d["r_pay"]], dev(d["s_key"]), [dev(x) for x in d["s_pay"]],
                      mat=mat, algo="phj", lds_budget=budget, radix_bits=bits)
    got = [host(k)] + [host(x) for x in r + s]
    want = oracle.join(d["r_key"], d["r_pay"], d["s_key"], d["s_pay"])
    order = np.argsort(want[0].astype(np.int64) & ((1 << bits) - 1), kind="stable")
    assert len(got[0]) == len(order) == n_s + hit * (extra > 0)
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a, np.asarray(b)[order])


@pytest.mark.parametrize("mat", ["gftr", "gfur"])
@pytest.mark.parametrize("cols", [1, 3])
def test_plan_of_mixed_instances(cols, mat):
    """Instances without, with one and with many S rows of several matches."""
    import paper_2312_00720_amd as gj
    from gpu_util import canon, dev, host, say
    say(f"join write paths, plan, {cols} columns {mat}")
    sizes = [(900, 5000, 0, 0), (3000, 20000, 1, 1), (50, 90, 5, 40), (2500, 9000, 800, 4000), (2, 3, 0, 0)]
    parts = [_data(*z, 4, cols, cols, seed=40 + i) for i, z in enumerate(sizes)]
    cat = lambda f: np.concatenate([f(p) for p in parts])
    off = lambda key: [0] + list(np.cumsum([len(p[key]) for p in parts]))
    plan = gj.JoinPlan(dev(cat(lambda p: p["r_key"])), [dev(cat(lambda p: p["r_pay"][j])) for j in range(cols)], off("r_key"),
                       dev(cat(lambda p: p["s_key"])), [dev(cat(lambda p: p["s_pay"][j])) for j in range(cols)], off("s_key"),
                       mat=mat, out_capacity=2 * sum(len(p["s_key"]) for p in parts))
    plan.run()
    k, r, s, o = plan.result()
    for i, p in enumerate(parts):
        lo, hi = int(o[i]), int(o[i + 1])
        got = canon([host(x)[lo:hi] for x in [k, *r, *s]])
        want = canon(oracle.join(p["r_key"], p["r_pay"], p["s_key"], p["s_pay"]))
        assert len(got[0]) == len(want[0])
        for a, b in zip(got, want):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("mat", ["gftr", "gfur"])
@pytest.mark.parametrize("kb,c_r,c_s,n_s", [(4, 2, 2, 3000), (8, 3, 1, 3000), (4, 1, 1, 3000), (4, 4, 4, 70000)])
def test_long_buckets(kb, c_r, c_s, n_s, mat):
    """Keys with 1 to 9, 63 to 65, 128 and 200 rows in one unit: rows written by a lane and
    by the wave, in one and in several steps of 64 entries, beside each other."""
    import paper_2312_00720_amd as gj
    from gpu_util import dev, host, say
    say(f"join long buckets {kb} {c_r} {c_s} {n_s} {mat}")
    g = datagen.rng(kb + n_s)
    reps = np.array([1, 2, 7, 8, 9, 63, 64, 65, 128, 200] + [1] * 300)
    keys = g.permutation(4 * len(reps))[:len(reps)].astype(np.int64)
    odd = 1 if kb == 4 else 0x5DEECE66D
    dt = np.int32 if kb == 4 else np.int64
    rk = (g.permutation(np.repeat(keys, reps)) * odd).astype(dt)
    few = g.integers(0, len(reps), size=n_s)
    few[g.random(n_s) < 0.9] = 20  # most S rows match one row, so that the result stays small
    sk = (np.where(g.random(n_s) < 0.3, 4 * len(reps) + 1, keys[few]) * odd).astype(dt)
    cols = lambda n, c: [g.integers(-2**62, 2**62, size=n, dtype=np.int64) if j % 2 == 1
                         else g.integers(-2**31, 2**31, size=n, dtype=np.int64).astype(np.int32) for j in range(c)]
    rp, sp = cols(len(rk), c_r), cols(n_s, c_s)
    k, r, s = gj.join(dev(rk), [dev(x) for x in rp], dev(sk), [dev(x) for x in sp], mat=mat, algo="phj", radix_bits=1)
    got = [host(k)] + [host(x) for x in r + s]
    want = oracle.join(rk, rp, sk, sp)
    order = np.argsort(want[0].astype(np.int64) & 1, kind="stable")
    assert len(got[0]) == len(order) > 0
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a, np.asarray(b)[order])
