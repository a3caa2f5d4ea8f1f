"""GPU parity of large passes in forms that the other tests leave out: digits of the
order-preserving key (a radix sort's) with sorted and with negative keys, and a batch of
a few large, uneven instances, whose segments have digit bits of their own and one of
which is empty. The launch names tell that whole lines were written."""
import pytest

from test_gpu_scatter_lines import _digit, _keys

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kb,n4,n8,lo,bits,kind", [(32, 4, 0, 24, 8, "sorted"), (32, 4, 0, 24, 8, "any"),
                                                   (32, 2, 0, 28, 4, "skew"), (64, 0, 1, 57, 7, "any"),
                                                   (64, 1, 1, 57, 7, "sorted")])
def test_ordered_digits(kb, n4, n8, lo, bits, kind):
    import torch
    import paper_2312_00720_amd as gj
    row = kb // 8 + 4 * n4 + 8 * n8 + 4
    n = (1 << (29 if kb == 32 else 31)) // row + 7777
    print(f"ordered n={n} kb={kb} {n4}+{n8} {lo} {bits} {kind}", flush=True)
    key = _keys(n, torch.int32 if kb == 32 else torch.int64, kind, seed=n)
    cols = [torch.arange(n, device="cuda", dtype=torch.int32) * (2 * j + 3) for j in range(n4)]
    cols += [torch.arange(n, device="cuda", dtype=torch.int64) * 5 - 7 for j in range(n8)]
    gj.profile_start()
    k, c, r, off = gj.partition(key, cols, bit_lo=lo, bits=bits, mode="ordered", rowid=True)
    torch.cuda.synchronize()
    assert gj.profile_stop()["k_hist_cells"]["launches"] == 1
    d = _digit(key, lo, bits, "ordered")
    perm = torch.sort(d, stable=True).indices
    count = torch.bincount(d, minlength=1 << bits)
    assert torch.equal(off, torch.cat([count.new_zeros(1), torch.cumsum(count, 0)]).to(torch.int32))
    assert torch.equal(k, key[perm]) and torch.equal(r, perm.to(torch.int32))
    for a, b in zip(c, cols):
        assert torch.equal(a, b[perm])


def test_batch_of_uneven_instances():
    """45 M, no, 20 M, 1000 and 77 rows a side: long chunks over segments of 8 bits and fewer."""
    import torch
    import paper_2312_00720_amd as gj
    sizes = [45_000_001, 0, 20_000_003, 1000, 77]
    n = sum(sizes)
    assert n * 12 >= 1 << 29
    print(f"batch of {sizes}", flush=True)
    off = [0]
    for m in sizes:
        off.append(off[-1] + m)
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    inst = torch.repeat_interleave(torch.arange(len(sizes), device="cuda"), torch.tensor(sizes, device="cuda"))
    rk = torch.cat([torch.randperm(m, generator=g, device="cuda") for m in sizes]).to(torch.int32)
    sk = torch.cat([torch.randint(0, max(m, 1), (m,), generator=g, device="cuda") for m in sizes]).to(torch.int32)
    tag = lambda i, k: (k.to(torch.int64) * 31 + i * 1009).to(torch.int32)
    rp = [tag(inst, rk), rk * 3]
    sp = [torch.arange(n, device="cuda", dtype=torch.int32), sk * 5]
    gj.profile_start()
    key, r, s, o = gj.join_batch(rk, rp, off, sk, sp, off, mat="gftr")
    torch.cuda.synchronize()
    assert gj.profile_stop()["k_hist_cells"]["launches"] == 2
    assert [int(x) for x in o] == off  # every S row matches once
    row = s[0].to(torch.int64)
    assert torch.equal(torch.sort(row).values, torch.arange(n, device="cuda"))
    assert torch.equal(key, sk[row]) and torch.equal(s[1], key * 5) and torch.equal(r[1], key * 3)
    assert torch.equal(r[0], tag(inst[row], key))
    assert torch.equal(inst[row], inst)  # instances in order
