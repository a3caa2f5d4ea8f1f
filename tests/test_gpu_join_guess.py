"""Joins of small build blocks that may not guess: where the partitions' mean R rows come
near the build block, the count pass runs once, sized by the unit count."""
import numpy as np
import pytest

import datagen
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mat", ["gftr", "gfur"])
@pytest.mark.parametrize("n_r,bits", [(6553, 1), (6554, 1), (8192, 1), (20000, 1), (1, 1), (52500, 4), (60000, 4)])
def test_count_pass_runs_once(n_r, bits, mat):
    import torch
    import paper_2312_00720_amd as gj
    from gpu_util import canon, dev, host, say
    say(f"join guess {n_r} {bits} {mat}")
    n_s = 50001
    d = datagen.pk_fk_join(n_r, n_s, 1, 2, seed=datagen.seed_for(n_r, bits), match_ratio=0.75)
    cols = [dev(x) for x in (d["r_key"], *d["r_pay"], d["s_key"], *d["s_pay"])]
    gj.profile_start()
    k, r, s = gj.join(cols[0], cols[1:2], cols[2], cols[3:], mat=mat, algo="phj", radix_bits=bits)
    torch.cuda.synchronize()
    assert gj.profile_stop()["k_join_count"]["launches"] == 1
    want = oracle.join(d["r_key"], d["r_pay"], d["s_key"], d["s_pay"])
    for a, b in zip(canon([host(k)] + [host(x) for x in r + s]), canon(want)):
        np.testing.assert_array_equal(a, b)
