"""The rows that a hash group-by of few groups inserts ahead of the rest: all of a small
input, and of a large one more than 16 per group, so that a key of a skewed input
is hardly ever left to the full pass, whose workgroups would all look it up."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("key64", [False, True])
@pytest.mark.parametrize("groups", [1, 3, 15, 20, 200, 1000])
@pytest.mark.parametrize("n,least", [(1, 1), (2048, 2048), (2049, 256), (6000, 256), (262145, 1024), (1 << 24, 2048)])
def test_rows_ahead(n, least, groups, key64):
    """The first 256 rows hold one key only; the prefix, from the launches' bytes, is longer."""
    import torch
    import paper_2312_00720_amd as gj
    from gpu_util import dev, host, say
    say(f"hgb prefix n={n} groups={groups} key64={key64}")
    g = np.random.default_rng(n + groups)
    key = (g.integers(0, groups, size=n) * 977 - 5).astype(np.int64 if key64 else np.int32)
    key[:256] = -5
    val = g.integers(-2**31, 2**31, size=n).astype(np.int32)
    gj.profile_start()
    k, (c, s) = gj.groupby(dev(key), [dev(val)], [(0, "count"), (0, "sum")], algo="hash")
    torch.cuda.synchronize()
    p = gj.profile_stop()["k_hgb_insert"]
    row = 12 if key64 else 8
    prefix = p["alg_bytes"] / row - (n if p["launches"] == 2 else 0)
    assert max(least, min(n, 14 * min(groups, len(np.unique(key))))) <= prefix <= n
    uk, inv = np.unique(key, return_inverse=True)
    k, c, s = host(k), host(c), host(s)
    order = np.argsort(k)
    np.testing.assert_array_equal(k[order], uk)
    np.testing.assert_array_equal(c[order], np.bincount(inv))
    want = np.zeros(len(uk), np.int64)
    np.add.at(want, inv, val.astype(np.int64))
    np.testing.assert_array_equal(s[order], want)
