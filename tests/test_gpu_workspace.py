"""A plan's workspace (slice partials, packed operands): calls on any streams
take turns with it, without waiting on the host."""
import ctypes
import threading

import numpy as np
import pytest
import torch

import oracle
from paper_1503_06202_amd import Plan, _lib, vis_shape

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")

# sliced small arrays, the sliced channel kernel, the packed path
SHAPES = [(40, 3, 8192), (200, 2, 8192), (704, 2, 5504)]


def frames(N, F, T, count):
    g = torch.Generator(device=DEV).manual_seed(N)
    x = [torch.randint(0, 256, (T, F, N), generator=g, device=DEV, dtype=torch.uint8)
         for _ in range(count)]
    return x, [oracle.to_int32(oracle.correlate(a.cpu().numpy())) for a in x]


@pytest.mark.parametrize("N,F,T", SHAPES)
def test_per_thread_streams_take_turns(N, F, T):
    # hipStreamPerThread is one handle, and another stream in every thread
    per_thread, turns = ctypes.c_void_p(2), 24
    x, ref = frames(N, F, T, 2)
    out = [torch.empty((turns,) + vis_shape(N, F), dtype=torch.int32, device=DEV) for _ in x]
    torch.cuda.synchronize()
    lock, fail = threading.Condition(), []
    turn = [0]
    print(f"per-thread streams N={N} F={F} T={T}", flush=True)
    with Plan(N, F, T) as p:

        def work(k):
            try:
                torch.cuda.set_device(0)
                for r in range(turns):
                    with lock:  # one call at a time, the threads in turn
                        assert lock.wait_for(lambda: turn[0] % 2 == k or fail, 60) and not fail
                        rc = _lib.lib().xeng_correlate(p.handle, x[k].data_ptr(), N, F, T,
                                                       out[k][r].data_ptr(), per_thread)
                        assert rc == _lib.XENG_OK, rc
                        turn[0] += 1
                        lock.notify_all()
                # a thread's stream ends with it, and events of work left there with the stream
                torch.cuda.ExternalStream(2).synchronize()
            except BaseException as err:  # reported by the main thread
                with lock:
                    fail.append(err)
                    lock.notify_all()

        threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        torch.cuda.synchronize()
    assert not fail, fail
    for k in range(2):
        got = out[k].cpu().numpy()
        for r in range(turns):
            assert np.array_equal(got[r], ref[k]), (k, r)


@pytest.mark.parametrize("first", ["null", "side"])
@pytest.mark.parametrize("N,F,T", SHAPES)
def test_second_stream_does_not_wait_on_the_host(N, F, T, first):
    x, ref = frames(N, F, T, 2)
    vis = [torch.empty(vis_shape(N, F), dtype=torch.int32, device=DEV) for _ in range(3)]
    a = torch.randn((8192, 8192), device=DEV, dtype=torch.bfloat16)
    s1 = torch.cuda.default_stream() if first == "null" else torch.cuda.Stream()
    s2, done = torch.cuda.Stream(), torch.cuda.Event()
    print(f"second stream N={N} F={F} T={T} {first}", flush=True)
    with Plan(N, F, T) as p:
        p.correlate(x[0], vis[0], stream=s1)
        b = a @ a
        torch.cuda.synchronize()
        with torch.cuda.stream(s1):
            for _ in range(100):  # about 0.1 s
                torch.mm(a, a, out=b)
            p.correlate(x[0], vis[0])
            done.record()
        p.correlate(x[1], vis[1], stream=s2)
        waited = done.query()
        p.correlate(x[0], vis[2], stream=s1)
        torch.cuda.synchronize()
    assert not waited
    for v, k in zip(vis, (0, 1, 0)):
        assert np.array_equal(v.cpu().numpy(), ref[k])


@pytest.mark.parametrize("N,F,T", SHAPES)
def test_first_and_growing_calls_beside_a_capture(N, F, T):
    # calls on a stream of their own, which allocate, while another is captured
    x, ref = frames(N, F, T, 1)
    half = x[0][:T // 2]
    ref_half = oracle.to_int32(oracle.correlate(half.cpu().numpy()))
    vis = [torch.zeros(vis_shape(N, F), dtype=torch.int32, device=DEV) for _ in range(5)]
    a, b, other = torch.ones(64, device=DEV), torch.zeros(64, device=DEV), torch.cuda.Stream()
    torch.cuda.synchronize()
    print(f"beside a capture N={N} F={F} T={T}", flush=True)
    with Plan(N, F, T) as p, Plan(N, F, T) as q, Plan(N, F, T) as r:
        q.correlate(half, vis[2], stream=other)  # its workspace grows below
        r.correlate(half, vis[3])  # on the null stream, then beside the capture
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            b.add_(a)
            p.correlate(x[0], vis[0], stream=other)
            q.correlate(x[0], vis[1], stream=other)
            r.correlate(x[0], vis[4], stream=other)
        for k in range(1, 4):
            g.replay()
            torch.cuda.synchronize()
            assert (b == k).all()
    assert np.array_equal(vis[0].cpu().numpy(), ref[0])
    assert np.array_equal(vis[1].cpu().numpy(), ref[0])
    assert np.array_equal(vis[2].cpu().numpy(), ref_half)
    assert np.array_equal(vis[3].cpu().numpy(), ref_half)
    assert np.array_equal(vis[4].cpu().numpy(), ref[0])
