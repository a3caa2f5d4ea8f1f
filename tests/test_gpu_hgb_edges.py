"""Hash group-by at the edges of its launch rules: rows around one round of a
workgroup and one chunk per XCD, batches of rows that end in the middle, and group
counts on either side of what the insert kernels cache."""
import numpy as np
import pytest

import datagen

pytestmark = pytest.mark.gpu

AGGS = [(0, "count"), (0, "sum"), (0, "min"), (0, "max"), (1, "sum"), (1, "min"), (1, "max")]


@pytest.mark.parametrize("key64", [False, True])
@pytest.mark.parametrize("groups", [5, 300])
@pytest.mark.parametrize("n", [1, 63, 2047, 2048, 2049, 8191, 8193, 16384, 16385, 70001])
def test_rows_at_chunk_edges(n, groups, key64):
    _check(n, groups, key64)


@pytest.mark.parametrize("key64", [False, True])
@pytest.mark.parametrize("groups", [2500, 3600, 5500, 7000])
def test_groups_at_cache_edges(groups, key64):
    _check(150001, groups, key64)


def _check(n, groups, key64):
    import paper_2312_00720_amd as gj
    from gpu_util import dev, host, say
    say(f"hgb n={n} groups={groups} key64={key64}")
    g = datagen.rng(n * 7 + groups + key64)
    key = (g.integers(0, groups, size=n) * 977 - 1000).astype(np.int64 if key64 else np.int32)
    vals = [g.integers(-2**31, 2**31, size=n).astype(np.int32) for _ in range(2)]
    k, outs = gj.groupby(dev(key), [dev(v) for v in vals], AGGS, algo="hash")
    k, outs = host(k), [host(o) for o in outs]
    order = np.argsort(k, kind="stable")
    uk, inv = np.unique(key, return_inverse=True)
    np.testing.assert_array_equal(k[order], uk)
    for (c, op), o in zip(AGGS, outs):
        v = vals[c].astype(np.int64)
        if op == "count":
            want = np.bincount(inv)
        elif op == "sum":
            want = np.zeros(len(uk), np.int64)
            np.add.at(want, inv, v)
        else:
            want = np.full(len(uk), 2**31 - 1 if op == "min" else -2**31, np.int64)
            (np.minimum if op == "min" else np.maximum).at(want, inv, v)
        np.testing.assert_array_equal(o[order].astype(np.int64), want)
