"""GPU parity of the partition group-by's discovery at the partition sizes where its
path changes: 2048 rows (one read, rows keep their slots), 65536 rows (slices and a
merge). Group order is part of the check: first occurrence within a partition, or
ascending keys for merged ones; partitions by the key's hash."""
import numpy as np
import pytest

import datagen

pytestmark = pytest.mark.gpu

I32_MIN, I64_MIN = -2**31, -2**63


def _fmix32(x):
    x = x.astype(np.uint64) & np.uint64(0xFFFFFFFF)
    m = np.uint64(0xFFFFFFFF)
    x ^= x >> np.uint64(16)
    x = (x * np.uint64(0x85EBCA6B)) & m
    x ^= x >> np.uint64(13)
    x = (x * np.uint64(0xC2B2AE35)) & m
    return x ^ (x >> np.uint64(16))


def _digit(key, bits):
    u = key.astype(np.int64).view(np.uint64)
    if key.dtype == np.int64:
        u = u ^ (u >> np.uint64(32))
    return (_fmix32(u) & np.uint64((1 << bits) - 1)).astype(np.int64)


CASES = [(n, g, kb) for n in (1, 2, 2047, 2048, 2049, 4097) for g, kb in ((1, 4), (3000, 4), (50, 8), (3000, 8))]
CASES += [(65536, 700, 4), (65537, 700, 4), (140000, 3000, 8)]


@pytest.mark.parametrize("n,g,kb", CASES)
def test_groups_in_discovery_order(n, g, kb):
    import paper_2312_00720_amd as gj
    from gpu_util import dev, host, say
    say(f"pgb discover n={n} g={g} kb={kb}")
    r = datagen.rng(n + g + kb)
    # one of two digits takes every row, so a partition has exactly n rows
    pool = r.integers(-2**31, 2**31, size=8 * g + 64).astype(np.int32 if kb == 4 else np.int64)
    if kb == 8:
        pool = pool * np.int64(0x100000001) + 12345
    pool[0] = I32_MIN if kb == 4 else I64_MIN  # the tables' empty marker
    want_digit = _digit(pool[:1], 1)[0]
    pool = pool[_digit(pool, 1) == want_digit][:g]
    key = pool[r.integers(0, len(pool), size=n)]
    val = r.integers(-2**31, 2**31, size=n).astype(np.int32)
    k, aggs = gj.groupby(dev(key), [dev(val)], [(0, "count"), (0, "sum"), (0, "min"), (0, "max")], algo="partition",
                         radix_bits=1)
    uniq, first, inv = np.unique(key, return_index=True, return_inverse=True)
    order = np.argsort(first, kind="stable") if n <= 65536 else np.arange(len(uniq))
    cnt = np.bincount(inv)
    total = np.zeros(len(uniq), np.int64)
    np.add.at(total, inv, val.astype(np.int64))
    lo, hi = np.full(len(uniq), 2**31 - 1, np.int32), np.full(len(uniq), -2**31, np.int32)
    np.minimum.at(lo, inv, val)
    np.maximum.at(hi, inv, val)
    np.testing.assert_array_equal(host(k), uniq[order])
    for a, b in zip(aggs, (cnt, total, lo, hi)):
        np.testing.assert_array_equal(host(a), b[order])
