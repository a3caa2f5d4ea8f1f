"""Allocators with little room: a call on a few thousand rows asks for no block much
larger than its columns, and its scratch and outputs together stay near their size."""
import ctypes

import pytest

import datagen

pytestmark = pytest.mark.gpu

MOST = 64 * 1024  # largest block the allocator serves
ROOM = 288 * 1024  # and all it holds at a time


class SmallAllocator:
    def __init__(self, gj):
        import torch
        self.live, self.held, self.requests = {}, 0, 0

        def _alloc(nbytes, _ctx):
            self.requests += 1
            if nbytes > MOST or self.held + nbytes > ROOM:
                return None
            t = torch.empty(int(nbytes), dtype=torch.uint8, device="cuda")
            self.live[t.data_ptr()] = t
            self.held += int(nbytes)
            return t.data_ptr()

        def _free(ptr, _ctx):
            self.held -= self.live.pop(int(ptr or 0)).numel()

        self._a, self._f = gj._ALLOC_FN(_alloc), gj._FREE_FN(_free)
        self.struct = gj.Allocator(self._a, self._f, None)


def _column(alloc, ptr, dtype, n):
    import torch
    return alloc.live[int(ptr)][:n * torch.empty(0, dtype=dtype).element_size()].view(dtype)


@pytest.mark.parametrize("mat", [1, 2])
@pytest.mark.parametrize("algo", [1, 2])
@pytest.mark.parametrize("n_r,n_s", [(1, 1), (40, 90), (1000, 4000)])
def test_join(n_r, n_s, algo, mat):
    import torch
    import paper_2312_00720_amd as gj
    from gpu_util import dev
    print(f"small allocator join {n_r} x {n_s} algo={algo} mat={mat}", flush=True)
    d = datagen.pk_fk_join(n_r, n_s, 1, 1, seed=datagen.seed_for(0, 91), match_ratio=1.0)
    rk, sk, rp, sp = dev(d["r_key"]), dev(d["s_key"]), dev(d["r_pay"][0]), dev(d["s_pay"][0])
    R = gj.Rel(gj._col(rk), (gj.Col * 1)(gj._col(rp)), 1, n_r)
    S = gj.Rel(gj._col(sk), (gj.Col * 1)(gj._col(sp)), 1, n_s)
    a = SmallAllocator(gj)
    ro, so = (ctypes.c_void_p * 1)(), (ctypes.c_void_p * 1)()
    out = gj.JoinOut(None, ro, so, 0)
    o = gj.JoinOpts(mat, 0, 0, 0, 0, 0.0, 0, 0, algo)
    rc = gj.lib().gj_join(ctypes.byref(R), ctypes.byref(S), ctypes.byref(o), ctypes.byref(a.struct),
                          gj._stream(rk.device), ctypes.byref(out))
    assert rc == 0, gj.lib().gj_last_error()
    assert out.n_rows == n_s and len(a.live) == 3
    key, s = _column(a, out.key, torch.int32, n_s), _column(a, so[0], torch.int32, n_s)
    order = torch.argsort(sk.to(torch.int64) * (1 << 32) + (sp.to(torch.int64) & 0xFFFFFFFF))
    got = torch.argsort(key.to(torch.int64) * (1 << 32) + (s.to(torch.int64) & 0xFFFFFFFF))
    assert torch.equal(key[got], sk[order]) and torch.equal(s[got], sp[order])


@pytest.mark.parametrize("algo", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("n", [1, 3000])
def test_group_by(n, algo):
    import torch
    import paper_2312_00720_amd as gj
    print(f"small allocator group-by n={n} algo={algo}", flush=True)
    key = torch.arange(n, device="cuda", dtype=torch.int32) % 70
    val = torch.arange(n, device="cuda", dtype=torch.int32)
    vp, ag = (gj.Col * 1)(gj._col(val)), (gj.Agg * 2)(gj.Agg(0, 2), gj.Agg(0, 1))
    a = SmallAllocator(gj)
    ao = (ctypes.c_void_p * 2)()
    out = gj.GroupByOut(None, ao, 0)
    o = gj.GroupByOpts(algo, 0, 0, 0, 0.0, 0, 0.0)
    rc = gj.lib().gj_groupby(gj._col(key), vp, 1, n, ag, 2, ctypes.byref(o), ctypes.byref(a.struct),
                             gj._stream(key.device), ctypes.byref(out))
    assert rc == 0, gj.lib().gj_last_error()
    g = min(n, 70)
    assert out.n_groups == g and len(a.live) == 3
    k = _column(a, out.key, torch.int32, g)
    order = torch.argsort(k)
    want = torch.zeros(g, dtype=torch.int64, device="cuda").index_add_(0, key.to(torch.int64), val.to(torch.int64))
    assert torch.equal(k[order], torch.arange(g, device="cuda", dtype=torch.int32))
    assert torch.equal(_column(a, ao[0], torch.int64, g)[order], torch.bincount(key, minlength=g))
    assert torch.equal(_column(a, ao[1], torch.int64, g)[order], want)


@pytest.mark.parametrize("bits", [5, 12])
def test_partition(bits):
    import torch
    import paper_2312_00720_amd as gj
    n = 3000
    print(f"small allocator partition bits={bits}", flush=True)
    key = torch.arange(n, device="cuda", dtype=torch.int32) * 2654435
    ok = torch.empty_like(key)
    a = SmallAllocator(gj)
    rc = gj.lib().gj_partition(gj._col(key), None, 0, n, 0, bits, 0, 0, ok.data_ptr(), None, None, None,
                               ctypes.byref(a.struct), gj._stream(key.device))
    assert rc == 0 and not a.live, gj.lib().gj_last_error()
    assert torch.equal(ok, key[torch.sort(key & ((1 << bits) - 1), stable=True).indices])
