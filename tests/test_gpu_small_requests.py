"""Small joins ask their allocator for one block of shared scratch beside the outputs, no
larger than the pieces of scratch that the call takes."""
import ctypes

import pytest

import datagen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_r,n_s", [(1, 4), (500, 2000), (1000, 4000)])
def test_join_takes_one_block(n_r, n_s):
    import torch
    import paper_2312_00720_amd as gj
    from gpu_util import dev
    print(f"small requests join {n_r} x {n_s}", flush=True)
    d = datagen.pk_fk_join(n_r, n_s, 1, 1, seed=datagen.seed_for(0, 93))
    rk, sk, rp, sp = dev(d["r_key"]), dev(d["s_key"]), dev(d["r_pay"][0]), dev(d["s_pay"][0])
    live, sizes = {}, []

    def alloc(nbytes, _ctx):
        t = torch.empty(int(nbytes), dtype=torch.uint8, device="cuda")
        live[t.data_ptr()] = t
        sizes.append(int(nbytes))
        return t.data_ptr()

    def free(ptr, _ctx):
        del live[int(ptr or 0)]

    a, f = gj._ALLOC_FN(alloc), gj._FREE_FN(free)
    st = gj.Allocator(a, f, None)
    R = gj.Rel(gj._col(rk), (gj.Col * 1)(gj._col(rp)), 1, n_r)
    S = gj.Rel(gj._col(sk), (gj.Col * 1)(gj._col(sp)), 1, n_s)
    ro, so = (ctypes.c_void_p * 1)(), (ctypes.c_void_p * 1)()
    out = gj.JoinOut(None, ro, so, 0)
    o = gj.JoinOpts(1, 0, 0, 0, 0, 0.0, 0, 0, 1)
    rc = gj.lib().gj_join(ctypes.byref(R), ctypes.byref(S), ctypes.byref(o), ctypes.byref(st),
                          gj._stream(rk.device), ctypes.byref(out))
    assert rc == 0 and out.n_rows == n_s and len(live) == 3
    up = lambda b: -(-b // 256) * 256
    outputs = 3 * up(4 * n_s)
    assert len(sizes) == 4 and sum(sizes) <= outputs + 8 * (n_r + n_s) + 2 * n_s + 20 * 256 + 256
    key = live[int(out.key)].cpu().numpy()[:4 * n_s].view("<i4")
    assert sorted(key.tolist()) == sorted(d["s_key"].tolist())
