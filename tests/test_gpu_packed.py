"""The packed path (frames of more than 640 inputs: samples repacked once into
FP6 operands, then 256 x 128 tiles) against the CPU oracle, bit-exact.

An FP6 e2m3 number holds a 4-bit code exactly, and the f32 sums of products of
codes stay integers below 450 x 32768 < 2^24 (over 64), so every result is
exact: no tolerance.  The shapes cover complete and partial fragments (32
inputs), blocks (128) and macro rows (256, odd block counts included), samples
that fill no step, round or sum block, the time slices' partial blocks, whole
rounds with a sliced tail, unaligned frames, segments of 32768 samples and the
largest sums.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1503_06202_amd import Plan, vis_shape

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def want(samples):
    return oracle.to_int32(oracle.correlate(samples))


def rand_frame(seed, T, F, N):
    return np.random.default_rng(seed).integers(0, 256, (T, F, N), dtype=np.uint8)


def gpu(samples, form="i8", vis=None, accumulate=False, split_t=0):
    T, F, N = samples.shape
    d = torch.from_numpy(np.ascontiguousarray(samples)).to(DEV)
    with Plan(N, F, T, form=form, accumulate=accumulate, split_t=split_t) as p:
        out = p.correlate(d, vis)
        torch.cuda.synchronize()
    return out.cpu().numpy()


# N x T, F such that the packed path is chosen (230,000 tile-samples)
SHAPES = [(641, 10961, 1), (704, 5504, 2), (768, 11008, 1), (769, 8300, 1), (897, 4233, 2),
          (1025, 5249, 1), (1090, 1537, 4), (1152, 5200, 1), (1281, 3600, 1), (2048, 1792, 1)]


@pytest.mark.parametrize("form", ["i8", "f8"])
@pytest.mark.parametrize("N,T,F", SHAPES)
def test_packed_shapes(N, T, F, form):
    s = rand_frame(N * 31 + T, T, F, N)
    print(f"packed N={N} F={F} T={T} form={form}", flush=True)
    assert np.array_equal(gpu(s, form), want(s))


@pytest.mark.parametrize("split", [1, 2, 3, 7])
def test_packed_slices_and_accumulate(split):
    s = rand_frame(5 + split, 5600, 2, 700)
    ref = want(s)
    assert np.array_equal(gpu(s, split_t=split), ref)
    base = np.random.default_rng(1).integers(-1000, 1000, ref.shape, dtype=np.int32)
    got = gpu(s, split_t=split, vis=torch.from_numpy(base).to(DEV), accumulate=True)
    assert np.array_equal(got, ref + base)


@pytest.mark.parametrize("accumulate", [False, True])
def test_packed_whole_rounds_and_tail(accumulate):
    # 36 tiles a channel, 8 channels: one round of 256 compute units and 32
    # tiles left for slices
    s = rand_frame(11, 2304, 8, 1536)
    ref = want(s)
    base = np.full(ref.shape, 7, np.int32)
    got = gpu(s, vis=torch.from_numpy(base).to(DEV), accumulate=accumulate)
    assert np.array_equal(got, ref + 7 if accumulate else ref)


def test_packed_segments():
    # 32768 samples a segment; the second one adds
    s = rand_frame(12, 32768 + 3 * 64 + 5, 1, 650)
    assert np.array_equal(gpu(s), want(s))


def test_packed_extreme_codes():
    # the largest sums of codes over one segment, in every accumulator kind
    T, N = 32768, 660
    for s in (np.full((T, 1, N), 0xFF, np.uint8), np.zeros((T, 1, N), np.uint8)):
        assert np.array_equal(gpu(s), want(s))
    r = np.random.default_rng(3)
    # real and imaginary codes 0 or 15, mostly 15: sums near the limit that
    # differ in their last bits
    hi = np.where(r.random((T, 1, N)) < 0.99, 0xF0, 0x00) | np.where(r.random((T, 1, N)) < 0.99, 15, 0)
    s = hi.astype(np.uint8)
    s[:, :, ::7] ^= (r.random((T, 1, len(range(0, N, 7)))) < 0.01).astype(np.uint8)
    assert np.array_equal(gpu(s), want(s))


@pytest.mark.parametrize("offset", [1, 8])
def test_packed_unaligned_frame_and_vis(offset):
    # samples at an odd byte, vis 4-byte but not 8-byte aligned, guards around both
    T, F, N = 5504, 2, 720
    s = rand_frame(21, T, F, N)
    raw = torch.full((s.size + 64,), 0x5A, dtype=torch.uint8, device=DEV)
    view = raw[offset:offset + s.size].view(T, F, N)
    view.copy_(torch.from_numpy(s).to(DEV))
    n = F * N * (N + 1)
    buf = torch.full((n + 64,), -77, dtype=torch.int32, device=DEV)
    vis = buf[33:33 + n].view(vis_shape(N, F))
    with Plan(N, F, T) as p:
        p.correlate(view, vis)
        torch.cuda.synchronize()
    assert np.array_equal(vis.cpu().numpy(), want(s))
    h = buf.cpu().numpy()
    assert (h[:33] == -77).all() and (h[33 + n:] == -77).all()
    assert (raw[:offset].cpu().numpy() == 0x5A).all()
    assert (raw[offset + s.size:].cpu().numpy() == 0x5A).all()


@pytest.mark.parametrize("step", [16, 128])
@pytest.mark.parametrize("N", [700, 768])
def test_packed_delays(N, step):
    # delays per 16 inputs, and equal within every block of 128
    D, T, F = 300, 5600, 2
    ext = rand_frame(31 + N, D + T, F, N)
    r = np.random.default_rng(N + step)
    d = np.repeat(r.integers(0, D + 1, (N + step - 1) // step), step)[:N].astype(np.int32)
    d[:step] = 0
    dev = torch.from_numpy(ext).to(DEV)
    with Plan(N, F, T) as p:
        p.set_delays(d, D)
        got = p.correlate(dev[D:])
        torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), oracle.to_int32(oracle.correlate_shifted(ext, D, d)))


# delays per 16 inputs take the packed path from 128 inputs on (340,000
# tile-samples); windows of the source meet the steps at every offset
@pytest.mark.parametrize("N,F,T,D", [(128, 60, 6011, 1), (144, 16, 7200, 31), (200, 16, 7111, 33),
                                     (300, 4, 14400, 2500), (656, 1, 33000, 20000)])
def test_packed_group_delays(N, F, T, D):
    ext = rand_frame(N + D, D + T, F, N)
    r = np.random.default_rng(N)
    d = np.repeat(r.integers(0, D + 1, (N + 15) // 16), 16)[:N].astype(np.int32)
    d[:16], d[16:32] = 0, D
    dev = torch.from_numpy(ext).to(DEV)
    ref = oracle.to_int32(oracle.correlate_shifted(ext, D, d))
    with Plan(N, F, T) as p:
        p.set_delays(d, D)
        assert np.array_equal(p.correlate(dev[D:]).cpu().numpy(), ref)
        p.set_delays(None)  # off again, on the same workspace
        assert np.array_equal(p.correlate(dev[D:].contiguous()).cpu().numpy(), want(ext[D:]))


def test_packed_workspace_orders_streams_and_grows():
    N = 700
    a, b, c = (rand_frame(40 + k, T, 2, N) for k, T in enumerate((5504, 5504, 9000)))
    da, db, dc = (torch.from_numpy(x).to(DEV) for x in (a, b, c))
    with Plan(N, 2, 9000) as p:
        s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
        v = [torch.empty(vis_shape(N, 2), dtype=torch.int32, device=DEV) for _ in range(3)]
        torch.cuda.synchronize()
        for _ in range(3):
            p.correlate(da, v[0], stream=s1)
            p.correlate(db, v[1], stream=s2)
        p.correlate(dc, v[2], stream=s1)  # longer: the workspace grows
        torch.cuda.synchronize()
    for x, y in zip((a, b, c), v):
        assert np.array_equal(y.cpu().numpy(), want(x))


def test_captured_call_equals_eager():
    # under capture the call takes kernels without plan-owned workspace; eager
    # calls between the replays use the workspace
    N, F, T = 704, 2, 5504
    x, y = rand_frame(50, T, F, N), rand_frame(51, T, F, N)
    d, e = torch.from_numpy(x).to(DEV), torch.from_numpy(y).to(DEV)
    vis = torch.zeros(vis_shape(N, F), dtype=torch.int32, device=DEV)
    with Plan(N, F, T) as p:
        p.correlate(d)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            p.correlate(d, vis)
        for src in (x, y, x):
            d.copy_(torch.from_numpy(src))
            vis.zero_()
            g.replay()
            other = p.correlate(e)
            torch.cuda.synchronize()
            assert np.array_equal(vis.cpu().numpy(), want(src))
            assert np.array_equal(other.cpu().numpy(), want(y))
        del g


@pytest.mark.parametrize("form", ["i8", "f8"])
@pytest.mark.parametrize("N,T,F", [(1100, 32768 + 3 * 64 + 5, 1),  # two segments, an odd block count
                                   (1090, 2049, 4), (2048, 2048, 4),  # short frames
                                   (641, 7001, 6)])
def test_packed_segments_and_short_frames(N, T, F, form):
    s = rand_frame(N + T, T, F, N)
    print(f"packed N={N} F={F} T={T} form={form}", flush=True)
    assert np.array_equal(gpu(s, form), want(s))


@pytest.mark.parametrize("N,F,T,D", [(144, 60, 6011, 31), (650, 2, 33000, 20000),
                                     (1040, 1, 33000, 300), (704, 3, 5600, 300), (768, 2, 5600, 300)])
def test_packed_group_delays_in_odd_blocks_and_segments(N, F, T, D):
    print(f"group delays N={N} F={F} T={T} D={D}", flush=True)
    test_packed_group_delays(N, F, T, D)
