"""GPU parity of joins whose S rows match several R rows, element by element: with
one build block per partition the rows come out by the key's partition, then in S
order, then in R order. Match counts on both sides of the chain sort's limit (32
rows in a bucket), of a wave's 256 output rows per step, and payload columns that do and do not
fit beside the table in LDS."""
import numpy as np
import pytest

import datagen
import oracle

pytestmark = pytest.mark.gpu


def _data(dup, distinct, n_s, kb, c_r, c_s, seed):
    g = datagen.rng(seed)
    dt = np.int32 if kb == 4 else np.int64
    keys = g.permutation(4 * distinct)[:distinct].astype(np.int64) * (1 if kb == 4 else 0x100000001)
    rk = g.permutation(np.repeat(keys, dup)).astype(dt)
    sk = np.concatenate([keys, g.integers(0, 4 * distinct, size=n_s - distinct)]).astype(dt)
    sk = g.permutation(sk)
    wide = lambda n, c: [g.integers(-2**62, 2**62, size=n, dtype=np.int64) if j % 3 == 2
                         else g.integers(-2**31, 2**31, size=n, dtype=np.int64).astype(np.int32) for j in range(c)]
    return {"r_key": rk, "r_pay": wide(len(rk), c_r), "s_key": sk, "s_pay": wide(len(sk), c_s)}


CASES = [
    # rows per key, distinct keys, S rows, key bytes, R / S payloads, lds_budget, radix_bits
    (2, 1000, 3001, 4, 1, 1, 0, 1),
    (31, 60, 500, 4, 2, 3, 0, 1),
    (32, 60, 500, 8, 2, 3, 0, 1),
    (33, 60, 500, 4, 2, 3, 0, 1),        # longer chains than the sort takes
    (200, 11, 130, 8, 8, 1, 0, 1),
    (4, 3000, 9000, 4, 8, 2, 8192, 1),   # eight R columns: the last ones stay in global memory
    (5, 5000, 20000, 4, 3, 1, 16384, 1),
    (3, 2500, 5000, 8, 4, 4, 8192, 1),
]


@pytest.mark.parametrize("mat", ["gftr", "gfur"])
@pytest.mark.parametrize("case", CASES)
def test_many_matches_element_by_element(case, mat):
    import paper_2312_00720_amd as gj
    from gpu_util import dev, host, say
    dup, distinct, n_s, kb, c_r, c_s, budget, bits = case
    say(f"join dups {case} {mat}")
    d = _data(dup, distinct, n_s, kb, c_r, c_s, seed=7000 + dup + kb)
    k, r, s = gj.join(dev(d["r_key"]), [dev(x) for x in d["r_pay"]], dev(d["s_key"]), [dev(x) for x in d["s_pay"]],
                      mat=mat, algo="phj", lds_budget=budget, radix_bits=bits)
    got = [host(k)] + [host(x) for x in r + s]
    want = oracle.join(d["r_key"], d["r_pay"], d["s_key"], d["s_pay"])
    order = np.argsort(want[0].astype(np.int64) & ((1 << bits) - 1), kind="stable")
    assert len(got[0]) == len(order) and len(order) > 0
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a, np.asarray(b)[order])


@pytest.mark.parametrize("big", [1300, 1700, 3500, 4500, 9000])
@pytest.mark.parametrize("mat", ["gftr", "gfur"])
def test_uneven_partitions(big, mat):
    """One R partition of `big` rows among sixteen of about 1200: within the LDS the
    count pass guesses, past it, past a build block, and past the spread limit
    (then both sides are partitioned on hashed keys)."""
    import paper_2312_00720_amd as gj
    from gpu_util import canon, dev, host, say
    say(f"join uneven big={big} {mat}")
    g = datagen.rng(big)
    n_r, n_s, bits = 20000, 70001, 4
    rest = n_r - big
    rk = np.concatenate([np.arange(big) * 16 + 3, np.arange(rest) // 15 * 16 + np.array([d for d in range(16) if d != 3])[np.arange(rest) % 15]])
    rk = g.permutation(rk).astype(np.int32)
    sk = g.integers(0, 16 * big, size=n_s).astype(np.int32)
    d = {"r_key": rk, "r_pay": datagen.payload_columns(g, n_r, 2), "s_key": sk, "s_pay": datagen.payload_columns(g, n_s, 2)}
    k, r, s = gj.join(dev(d["r_key"]), [dev(x) for x in d["r_pay"]], dev(d["s_key"]), [dev(x) for x in d["s_pay"]],
                      mat=mat, algo="phj")
    got = [host(k)] + [host(x) for x in r + s]
    want = oracle.join(d["r_key"], d["r_pay"], d["s_key"], d["s_pay"])
    assert len(got[0]) == len(want[0])
    if big <= 4096:
        order = np.argsort(want[0] & ((1 << bits) - 1), kind="stable")
        for a, b in zip(got, want):
            np.testing.assert_array_equal(a, np.asarray(b)[order])
    else:
        for a, b in zip(canon(got), canon(want)):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("key64", [False, True])
@pytest.mark.parametrize("n_s", [131071, 131072, 496 * 8192, 496 * 8192 + 1])
def test_units_of_few_and_many_waves(n_s, key64):
    """16 partitions: units of 16 waves from 131072 S rows (4096 for each of 32 units)
    to 496 S pieces (512 units), of four on either side; some S rows match nothing,
    some R keys repeat."""
    import paper_2312_00720_amd as gj
    from gpu_util import dev, host, say
    say(f"join waves n_s={n_s} key64={key64}")
    g = datagen.rng(n_s + key64)
    dt = np.int64 if key64 else np.int32
    rk = g.permutation(np.concatenate([np.arange(18000), np.arange(2000)])).astype(dt)
    sk = g.integers(0, 24000, size=n_s).astype(dt)
    rp, sp = datagen.payload_columns(g, len(rk), 1), datagen.payload_columns(g, n_s, 1)
    k, r, s = gj.join(dev(rk), [dev(x) for x in rp], dev(sk), [dev(x) for x in sp], mat="gftr", algo="phj")
    got = [host(k)] + [host(x) for x in r + s]
    want = oracle.join(rk, rp, sk, sp)
    assert len(got[0]) == len(want[0])
    order = np.argsort(want[0] & 15, kind="stable")
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a, np.asarray(b)[order])
