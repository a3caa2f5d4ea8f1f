"""GPU parity of partition passes at the sizes where their tiles change, for few and
many digit bits, both key widths, one and two passes, and a partition group-by, whose
tiles are those of an 8-bit pass whatever its digit bits."""
import pytest

from test_gpu_scatter_lines import _digit, _keys

pytestmark = pytest.mark.gpu

SIZES = [(1 << 20) + 1, (1 << 21) + 1, 5 << 19, (5 << 19) + 1, 1 << 22, (1 << 22) + 1, (11 << 19) + 1, (3 << 21) + 1]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("kb,bits,passes", [(32, 3, 1), (32, 8, 1), (64, 3, 1), (64, 8, 1), (32, 12, 2), (64, 11, 2)])
def test_partition(n, kb, bits, passes):
    import torch
    import paper_2312_00720_amd as gj
    print(f"tile edges n={n} kb={kb} bits={bits}/{passes}", flush=True)
    key = _keys(n, torch.int32 if kb == 32 else torch.int64, "any", seed=n + bits)
    cols = [torch.arange(n, device="cuda", dtype=torch.int32) * 3, torch.arange(n, device="cuda", dtype=torch.int64) - 7]
    k, c, r, off = gj.partition(key, cols, bits=bits, passes=passes, rowid=True)
    d = _digit(key, 0, bits, "bits")
    perm = torch.sort(d, stable=True).indices
    count = torch.bincount(d, minlength=1 << bits)
    assert torch.equal(off, torch.cat([count.new_zeros(1), torch.cumsum(count, 0)]).to(torch.int32))
    assert torch.equal(k, key[perm]) and torch.equal(r, perm.to(torch.int32))
    assert torch.equal(c[0], cols[0][perm]) and torch.equal(c[1], cols[1][perm])


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("groups,key64", [(20, False), (30000, False), (400, True)])
def test_group_by(n, groups, key64):
    import torch
    import paper_2312_00720_amd as gj
    print(f"tile edges group-by n={n} groups={groups}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(n + groups)
    idx = torch.randint(0, groups, (n,), generator=g, device="cuda")
    key = idx * 0x5DEECE66D if key64 else idx.to(torch.int32)
    val = torch.randint(-2 ** 20, 2 ** 20, (n,), generator=g, device="cuda", dtype=torch.int32)
    k, (cnt, tot) = gj.groupby(key, [val], [(0, "count"), (0, "sum")], algo="partition")
    order = torch.argsort(k)
    assert k.numel() == groups
    assert torch.equal(cnt[order], torch.bincount(idx, minlength=groups))
    want = torch.zeros(groups, dtype=torch.int64, device="cuda").index_add_(0, idx, val.to(torch.int64))
    assert torch.equal(tot[order], want)


@pytest.mark.parametrize("n,rows", [(1 << 20, 2048), ((1 << 20) + 1, 4096), (1 << 22, 4096), ((3 << 21) + 1, 16384)])
def test_sketch_chunks(n, rows):
    """8-byte keys: the sketch's workgroups count 4096 rows at least from 2^20 rows, from the bytes
    of the fold that follows them (256 counts in, 2^bits out for every chunk)."""
    import torch
    import paper_2312_00720_amd as gj
    print(f"sketch chunks n={n}", flush=True)
    idx = torch.arange(n, device="cuda") * 7919 % 400
    val = torch.arange(n, device="cuda", dtype=torch.int32)
    gj.profile_start()
    k, (cnt,) = gj.groupby(idx * 0x5DEECE66D, [val], [(0, "count")], algo="partition")
    torch.cuda.synchronize()
    p = gj.profile_stop()
    chunks = -(-n // rows)
    assert p["k_fold_hist"]["alg_bytes"] in [4.0 * chunks * (256 + (1 << b)) for b in range(1, 9)]
    assert torch.equal(cnt[torch.argsort(k)], torch.bincount(idx))
