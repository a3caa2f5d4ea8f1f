"""Calls from several threads on streams of their own: every call reads its counts
back through its thread's host block, so concurrent results equal the ones of calls
made alone."""
import threading

import pytest

pytestmark = pytest.mark.gpu


def _work(gj, torch, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    n_r, n_s = 3000 + 700 * seed, 20000 + 1111 * seed
    r = torch.randperm(n_r, generator=g, device="cuda").to(torch.int32)
    s = torch.randint(0, 2 * n_r, (n_s,), generator=g, device="cuda").to(torch.int32)
    return r, [r * 3], s, [s * 5]


def _call(gj, torch, cols):
    r, rp, s, sp = cols
    k, a, b = gj.join(r, rp, s, sp)
    gk, aggs = gj.groupby(s, sp, [(0, "count"), (0, "sum")], algo="partition")
    sk, smax = gj.groupby(s, sp, [(0, "max")], algo="sort")
    return [k, *a, *b, gk, *aggs, sk, *smax]


@pytest.mark.parametrize("threads", [2, 4])
def test_threads_on_their_own_streams(threads):
    import torch
    import paper_2312_00720_amd as gj
    print(f"{threads} threads", flush=True)
    cols = [_work(gj, torch, i) for i in range(threads)]
    alone = [_call(gj, torch, c) for c in cols]
    torch.cuda.synchronize()
    out, errors = [None] * threads, []

    def body(i):
        try:
            st = torch.cuda.Stream()
            with torch.cuda.stream(st):
                for _ in range(20):
                    out[i] = _call(gj, torch, cols[i])
                st.synchronize()
        except Exception as e:  # reported by the test's own thread
            errors.append((i, repr(e)))

    ts = [threading.Thread(target=body, args=(i,)) for i in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors, errors
    for a, b in zip(alone, out):
        assert len(a) == len(b)
        for x, y in zip(a, b):
            assert torch.equal(x, y)
