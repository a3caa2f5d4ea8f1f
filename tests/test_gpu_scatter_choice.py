"""GPU parity of large partition passes on either side of the choice between whole
lines over long chunks and the wide kernel over short ones, with the side taken read
from the launch names: digits of few bits, rows whose carry does not fit, outputs that
are not 16-byte aligned, two passes, and a partition group-by, whose chunks are fixed
before its digit bits are known."""
import pytest

from test_gpu_scatter_lines import _digit, _keys

pytestmark = pytest.mark.gpu


def _profiled(gj, torch, call):
    gj.profile_start()
    out = call()
    torch.cuda.synchronize()
    return out, gj.profile_stop()


CASES = [
    # key bits, 4-byte columns, 8-byte columns, row id, bit_lo, bits, passes, mode, keys, passes in long chunks
    (32, 2, 0, False, 0, 2, 1, "bits", "any", 0),
    (32, 4, 0, False, 0, 3, 1, "hash", "skew", 0),
    (32, 4, 0, False, 7, 4, 1, "bits", "any", 1),
    (32, 6, 0, False, 0, 8, 1, "bits", "any", 0),        # 28 bytes a row
    (32, 6, 0, True, 0, 15, 2, "bits", "any", 1),        # 8 bits, then 7 over segments
    (64, 0, 1, False, 0, 5, 1, "bits", "any", 0),
    (64, 0, 1, False, 0, 16, 2, "hash", "skew", 0),
    (64, 0, 1, False, 0, 14, 2, "bits", "any", 2),
]


@pytest.mark.parametrize("case", CASES)
def test_side_and_result(case):
    import torch
    import paper_2312_00720_amd as gj
    kb, n4, n8, rowid, lo, bits, passes, mode, kind, long_passes = case
    dt = torch.int32 if kb == 32 else torch.int64
    row = kb // 8 + 4 * n4 + 8 * n8 + (4 if rowid else 0)
    n = (1 << (29 if kb == 32 and n8 == 0 else 31)) // row + 54321
    print(f"choice n={n} {case}", flush=True)
    key = _keys(n, dt, kind, seed=n + bits)
    cols = [torch.arange(n, device="cuda", dtype=torch.int32) * (2 * j + 3) for j in range(n4)]
    cols += [torch.arange(n, device="cuda", dtype=torch.int64) * (2 * j + 5) - 7 for j in range(n8)]
    (k, c, r, off), prof = _profiled(gj, torch, lambda: gj.partition(key, cols, bit_lo=lo, bits=bits, passes=passes,
                                                                     mode=mode, rowid=rowid))
    assert prof.get("k_hist_cells", {"launches": 0})["launches"] == long_passes
    assert prof["k_scatter"]["launches"] == passes
    d = _digit(key, lo, bits, mode)
    perm = torch.sort(d, stable=True).indices
    count = torch.bincount(d, minlength=1 << bits)
    assert torch.equal(off, torch.cat([count.new_zeros(1), torch.cumsum(count, 0)]).to(torch.int32))
    assert torch.equal(k, key[perm])
    for a, b in zip(c, cols):
        assert torch.equal(a, b[perm])
    if rowid:
        assert torch.equal(r, perm.to(torch.int32))


def test_unaligned_outputs_take_short_chunks():
    import torch
    import paper_2312_00720_amd as gj
    n = (1 << 29) // 12 + 999
    print(f"choice unaligned n={n}", flush=True)
    key = _keys(n, torch.int32, "any", seed=5)
    cols = [torch.arange(n, device="cuda", dtype=torch.int32) * (2 * j + 3) for j in range(2)]
    out = [torch.empty(n + 4, device="cuda", dtype=torch.int32)[s:s + n] for s in (0, 4, 1)]
    off = torch.empty(129, device="cuda", dtype=torch.int32)
    _, prof = _profiled(gj, torch, lambda: gj.partition_noalloc(key, cols, out[0], out[1:], off, bits=7))
    assert "k_hist_cells" not in prof
    perm = torch.sort(_digit(key, 0, 7, "bits"), stable=True).indices
    for a, b in zip(out, [key, *cols]):
        assert torch.equal(a, b[perm])


@pytest.mark.parametrize("groups,n8,n4", [(20, 1, 0), (400, 1, 0), (400, 1, 1), (9000, 1, 0), (60000, 1, 1), (400, 0, 6)])
def test_group_by_counts_and_pass_agree(groups, n8, n4):
    """Rows of 12, 16 and 28 bytes, 4 to 8 digit bits: the sketch's chunks may not be
    those the pass would choose itself."""
    import torch
    import paper_2312_00720_amd as gj
    n = (1 << (31 if n8 else 29)) // (4 + 8 * n8 + 4 * n4) + 777
    print(f"choice group-by n={n} groups={groups} n8={n8} n4={n4}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(groups)
    key = torch.randint(0, groups, (n,), generator=g, device="cuda", dtype=torch.int32)
    vals = [torch.randint(-2 ** 20, 2 ** 20, (n,), generator=g, device="cuda", dtype=torch.int32) for _ in range(n4)]
    vals += [torch.randint(-2 ** 40, 2 ** 40, (n,), generator=g, device="cuda", dtype=torch.int64) for _ in range(n8)]
    aggs = [(0, "count")] + [(c, "sum") for c in range(len(vals))]
    k, out = gj.groupby(key, vals, aggs, algo="partition")
    order = torch.argsort(k)
    assert torch.equal(k[order], torch.arange(groups, device="cuda", dtype=torch.int32))
    idx = key.to(torch.int64)
    assert torch.equal(out[0][order], torch.bincount(idx, minlength=groups))
    for c, v in enumerate(vals):
        want = torch.zeros(groups, dtype=torch.int64, device="cuda").index_add_(0, idx, v.to(torch.int64))
        assert torch.equal(out[1 + c][order], want)
