"""Counts reach the host beside other work on the device: a thread that called the
library and ends does not wait for other streams; many threads share a few host blocks;
a plan's result asked for on one stream covers a run on the default stream."""
import os
import threading
import time

import pytest

pytestmark = pytest.mark.gpu


def _cols(torch):
    r = torch.randperm(3000, device="cuda").to(torch.int32)
    s = torch.randint(0, 3000, (9000,), device="cuda", dtype=torch.int32)
    return r, [r * 3], s, [s * 5]


def _in_thread(torch, gj, cols):
    """A join in a new thread on a stream of its own: columns, error, whether the thread ended."""
    out = [None, None]
    ident = []

    def body():
        ident.append(threading.get_native_id())
        try:
            st = torch.cuda.Stream()
            with torch.cuda.stream(st):
                k, r, s = gj.join(*cols)
                st.synchronize()
                out[0] = [k, *r, *s]
        except Exception as e:  # reported by the test's own thread
            out[1] = repr(e)

    t = threading.Thread(target=body)
    t.start()
    t.join()
    # gone with everything that is its own (Python's join only waits for its Python part)
    end = time.perf_counter() + 0.3
    while os.path.exists(f"/proc/self/task/{ident[0]}") and time.perf_counter() < end:
        time.sleep(0.002)
    out.append(not os.path.exists(f"/proc/self/task/{ident[0]}"))
    return out


def _check(torch, cols, got):
    k, r, s = got
    assert k.numel() == cols[2].numel()
    assert torch.equal(r, k * 3) and torch.equal(s, k * 5)
    assert torch.equal(torch.sort(k).values, torch.sort(cols[2]).values)


def _busy(torch, seconds):
    """About that long of work on the current stream."""
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    torch.cuda._sleep(10 ** 7)
    torch.cuda.synchronize()
    torch.cuda._sleep(int(10 ** 7 / (time.perf_counter() - t0) * seconds))


def test_ending_thread_does_not_wait_for_the_device():
    import torch
    import paper_2312_00720_amd as gj
    print("thread end beside a busy stream", flush=True)
    cols = _cols(torch)
    _in_thread(torch, gj, cols)
    done = torch.cuda.Event()
    _busy(torch, 1.0)
    done.record()
    got, err, ended = _in_thread(torch, gj, cols)
    busy = not done.query()
    torch.cuda.synchronize()
    assert err is None, err
    assert busy and ended
    _check(torch, cols, got)


def test_more_threads_than_blocks():
    import torch
    import paper_2312_00720_amd as gj
    print("24 threads at a time", flush=True)
    cols = _cols(torch)
    torch.cuda.synchronize()
    gate, out = threading.Barrier(24), []

    def body():
        try:
            st = torch.cuda.Stream()
            gate.wait()
            with torch.cuda.stream(st):
                for _ in range(5):
                    k, r, s = gj.join(*cols)
                st.synchronize()
            out.append([k, r[0], s[0]])
        except Exception as e:  # reported by the test's own thread
            out.append(repr(e))

    ts = [threading.Thread(target=body) for _ in range(24)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    assert not [x for x in out if isinstance(x, str)], out
    for got in out:
        _check(torch, cols, got)


@pytest.mark.parametrize("kind", ["join", "groupby"])
@pytest.mark.parametrize("graph", [False, True])
def test_plan_result_on_another_stream(kind, graph):
    import torch
    import paper_2312_00720_amd as gj
    print(f"plan result on another stream {kind} graph={graph}", flush=True)
    r, rp, s, sp = _cols(torch)
    if kind == "join":
        plan = gj.JoinPlan(r, rp, [0, 1000, 3000], s, sp, [0, 4000, 9000])
    else:
        plan = gj.GroupByPlan(s, sp, [0, 4000, 9000], [(0, "count"), (0, "sum")])
    if graph:
        plan.capture()
    side = torch.cuda.Stream()
    for _ in range(2):
        _busy(torch, 0.2)
        s.add_(1).remainder_(1700)  # other keys, other sizes
        plan.launch() if graph else plan.run()
        with torch.cuda.stream(side):
            got = plan.result()
            got = [x.clone() for x in ([got[0], *got[1]] if kind == "groupby" else [got[0], *got[1], *got[2]])] + [got[-1]]
            side.synchronize()
        plan.launch() if graph else plan.run()
        torch.cuda.synchronize()
        again = plan.result()
        again = ([again[0], *again[1]] if kind == "groupby" else [again[0], *again[1], *again[2]]) + [again[-1]]
        assert got[-1] == again[-1] and got[-1][-1] == got[0].numel()
        for a, b in zip(got[:-1], again[:-1]):
            assert torch.equal(a, b)
        if kind == "groupby":
            assert int(got[1].sum()) == s.numel()
