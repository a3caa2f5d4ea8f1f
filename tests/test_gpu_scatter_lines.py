"""GPU parity of the whole-line scatter, which large passes take (the radix-partition
primitive of Section 2.3): every output element against a stable sort by digit on the
device. Sizes just past the kernel's range with ragged tails; digits that fill whole
lines, that leave every line to the carry, and that put most rows in one digit; two
passes, whose chunks are cut by segments; outputs that are not 16-byte aligned."""
import pytest

pytestmark = pytest.mark.gpu


def _fmix32(x):
    m = 0xFFFFFFFF
    x = x ^ (x >> 16)
    x = (x * 0x85EBCA6B) & m
    x = x ^ (x >> 13)
    x = (x * 0xC2B2AE35) & m
    return x ^ (x >> 16)


def _digit(key, lo, bits, mode):
    import torch
    u = key.to(torch.int64)
    if mode == "hash":
        u = _fmix32(u & 0xFFFFFFFF if key.dtype == torch.int32 else (u ^ (u >> 32)) & 0xFFFFFFFF)
    elif mode == "ordered":
        u = u ^ (1 << 31 if key.dtype == torch.int32 else -(1 << 63))
    return (u >> lo) & ((1 << bits) - 1)


def _keys(n, dtype, kind, seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    if dtype == torch.int32:
        k = torch.randint(-2 ** 31, 2 ** 31 - 1, (n,), generator=g, device="cuda", dtype=torch.int32)
    else:
        k = torch.randint(-2 ** 62, 2 ** 62, (n,), generator=g, device="cuda", dtype=torch.int64)
    if kind == "one":       # a single digit value: one run across every tile
        k.fill_(5)
    elif kind == "skew":    # seven rows of eight in one digit, the rest anywhere
        k[torch.rand(n, generator=g, device="cuda") < 0.875] = 3
    elif kind == "sorted":  # long runs of equal digits
        k = torch.sort(k).values
    return k


CASES = [
    # key bits, 4-byte columns, 8-byte columns, row id, bit_lo, bits, passes, mode, keys
    (32, 4, 0, False, 0, 7, 1, "bits", "any"),
    (32, 4, 0, False, 3, 1, 1, "bits", "any"),
    (32, 4, 0, False, 0, 7, 1, "bits", "skew"),
    (32, 4, 0, False, 0, 7, 1, "bits", "one"),
    (32, 2, 0, False, 0, 8, 1, "hash", "any"),
    (32, 7, 0, True, 24, 8, 1, "ordered", "sorted"),   # 36 bytes a row: short tiles
    (32, 4, 0, False, 0, 13, 2, "bits", "any"),        # segments cut the chunks
    (32, 3, 0, True, 0, 16, 2, "hash", "skew"),
    (32, 1, 2, False, 0, 6, 1, "bits", "any"),
    (64, 2, 1, False, 0, 7, 1, "hash", "any"),
    (64, 1, 1, False, 5, 12, 2, "bits", "skew"),
    (64, 4, 4, True, 0, 8, 1, "bits", "any"),          # no room for the carry: the wide kernel
]


@pytest.mark.parametrize("case", CASES)
def test_large_pass_matches_stable_sort(case):
    import torch
    import paper_2312_00720_amd as gj
    kb, n4, n8, rowid, lo, bits, passes, mode, kind = case
    dt = torch.int32 if kb == 32 else torch.int64
    row = kb // 8 + 4 * n4 + 8 * n8 + (4 if rowid else 0)
    narrow = kb == 32 and n8 == 0
    n = (1 << (29 if narrow else 31)) // row + 12345
    print(f"large pass n={n} {case}", flush=True)
    key = _keys(n, dt, kind, seed=n + bits)
    cols = [torch.arange(n, device="cuda", dtype=torch.int32) * (2 * j + 3) for j in range(n4)]
    cols += [torch.arange(n, device="cuda", dtype=torch.int64) * (2 * j + 5) - 7 for j in range(n8)]
    k, c, r, off = gj.partition(key, cols, bit_lo=lo, bits=bits, passes=passes, mode=mode, rowid=rowid)
    d = _digit(key, lo, bits, mode)
    perm = torch.sort(d, stable=True).indices
    count = torch.bincount(d, minlength=1 << bits)
    want = torch.cat([count.new_zeros(1), torch.cumsum(count, 0)]).to(torch.int32)
    assert torch.equal(off, want)
    assert torch.equal(k, key[perm])
    for a, b in zip(c, cols):
        assert torch.equal(a, b[perm])
    if rowid:
        assert torch.equal(r, perm.to(torch.int32))


@pytest.mark.parametrize("shift", [0, 1, 3])
def test_large_pass_into_unaligned_outputs(shift):
    """Columns that start `shift` elements into their buffers, and nothing written before or after them."""
    import torch
    import paper_2312_00720_amd as gj
    n = (1 << 29) // 12 + 4321
    print(f"unaligned outputs n={n} shift={shift}", flush=True)
    key = _keys(n, torch.int32, "any", seed=77)
    cols = [torch.arange(n, device="cuda", dtype=torch.int32) * (2 * j + 3) for j in range(2)]
    room = [torch.full((n + 8,), -9, device="cuda", dtype=torch.int32) for _ in range(3)]
    out = [x[shift:shift + n] for x in room]
    off = torch.empty(129, device="cuda", dtype=torch.int32)
    gj.partition_noalloc(key, cols, out[0], out[1:], off, bits=7)
    perm = torch.sort(_digit(key, 0, 7, "bits"), stable=True).indices
    for a, b, x in zip(out, [key, *cols], room):
        assert torch.equal(a, b[perm])
        assert bool((x[:shift] == -9).all()) and bool((x[shift + n:] == -9).all())


PASS_CASES = [
    # n, bits, passes: one tile (no histogram), counts summed by the scatter, scanned by
    # one workgroup and by several; the shapes' and the second pass's boundaries
    (1, 8, 1), (2047, 3, 1), (2048, 8, 1), (2049, 8, 1),
    (131072, 8, 1), (131073, 8, 1), (300001, 5, 1), (1 << 20, 5, 1), ((1 << 20) + 1, 8, 1),
    ((3 << 21), 4, 1), ((3 << 21) + 1, 8, 1),
    (2049, 16, 2), (40000, 9, 2), (1 << 20, 12, 2), (1500001, 10, 2),
]


@pytest.mark.parametrize("n,bits,passes", PASS_CASES)
@pytest.mark.parametrize("kb,kind", [(32, "any"), (64, "skew")])
def test_pass_shapes_match_stable_sort(n, bits, passes, kb, kind):
    import torch
    import paper_2312_00720_amd as gj
    print(f"pass n={n} bits={bits} passes={passes} kb={kb} {kind}", flush=True)
    key = _keys(n, torch.int32 if kb == 32 else torch.int64, kind, seed=n + bits)
    if kind == "skew":
        key = key & 0x0F0F0F0F0F0F0F0F  # most segments of a second pass are empty
    cols = [torch.arange(n, device="cuda", dtype=torch.int32) * 3, torch.arange(n, device="cuda", dtype=torch.int64) - 7]
    k, c, r, off = gj.partition(key, cols, bits=bits, passes=passes, rowid=True)
    d = _digit(key, 0, bits, "bits")
    perm = torch.sort(d, stable=True).indices
    count = torch.bincount(d, minlength=1 << bits)
    assert torch.equal(off, torch.cat([count.new_zeros(1), torch.cumsum(count, 0)]).to(torch.int32))
    assert torch.equal(k, key[perm]) and torch.equal(r, perm.to(torch.int32))
    assert torch.equal(c[0], cols[0][perm]) and torch.equal(c[1], cols[1][perm])
