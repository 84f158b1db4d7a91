"""The small-array kernel (at most 128 inputs: several channels a workgroup)
against the CPU oracle, bit-exact, in both forms.

The shapes cover one input up to a full column set of every width (16, 32, 64,
128 columns a channel), channel counts that fill a workgroup partly and span
several, frames of part of a chunk up to more turns than a wave's loads ahead,
time slices (partial triangles summed by a second launch), accumulation,
unaligned frames and the integration limit of the int32 sums.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1503_06202_amd import Plan, vis_shape

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def rand_frame(seed, T, F, N):
    return np.random.default_rng(seed).integers(0, 256, (T, F, N), dtype=np.uint8)


def want(s):
    return oracle.to_int32(oracle.correlate(s))


def run(s, form="i8", split=0, vis=None, accumulate=False):
    T, F, N = s.shape
    d = torch.from_numpy(s).to(DEV)
    with Plan(N, F, T, form=form, split_t=split, accumulate=accumulate) as p:
        out = p.correlate(d, vis)
        torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("N,F", [(1, 1), (1, 9), (5, 8), (15, 3), (16, 8), (16, 17), (17, 4),
                                 (31, 5), (32, 4), (33, 2), (48, 3), (63, 1), (64, 2), (64, 5),
                                 (65, 1), (100, 2), (127, 1), (128, 3)])
@pytest.mark.parametrize("T", [1, 64, 130, 256, 1000])
def test_small_shapes(N, F, T):
    s = rand_frame(N * 1000 + F * 10 + T, T, F, N)
    ref = want(s)
    assert np.array_equal(run(s), ref)
    assert np.array_equal(run(s, form="f8"), ref)


@pytest.mark.parametrize("N,F", [(9, 11), (30, 6), (64, 3), (120, 2)])
@pytest.mark.parametrize("split", [0, 2, 5, 8, 33])
def test_small_slices_and_accumulate(N, F, split):
    s = rand_frame(N + split, 4096 + 77, F, N)
    ref = want(s)
    assert np.array_equal(run(s, split=split), ref)
    base = np.random.default_rng(2).integers(-5000, 5000, ref.shape, dtype=np.int32)
    got = run(s, split=split, vis=torch.from_numpy(base).to(DEV), accumulate=True)
    assert np.array_equal(got, ref + base)


@pytest.mark.parametrize("N", [16, 64, 128])
def test_small_unaligned_vis_and_guards(N):
    # vis 4-byte aligned (the slice sum by single ints), guards around both buffers
    T, F = 2048, 5
    s = rand_frame(N, T, F, N)
    n = F * N * (N + 1)
    for split in (1, 4):
        buf = torch.full((n + 64,), -77, dtype=torch.int32, device=DEV)
        vis = buf[33:33 + n].view(vis_shape(N, F))
        with Plan(N, F, T, split_t=split) as p:
            p.correlate(torch.from_numpy(s).to(DEV), vis)
            torch.cuda.synchronize()
        assert np.array_equal(vis.cpu().numpy(), want(s))
        h = buf.cpu().numpy()
        assert (h[:33] == -77).all() and (h[33 + n:] == -77).all()


@pytest.mark.parametrize("N", [3, 40, 72])
def test_small_integration_limit(N):
    # 2^19 samples a launch (the next one adds), extreme codes on both sides
    T = (1 << 19) + 3 * 64 + 5
    s = np.where(np.arange(N)[None, None, :] % 2 == 0, 0x00, 0xFF).astype(np.uint8)
    s = np.broadcast_to(s, (T, 1, N)).copy()
    s[::3] ^= 0x0F
    ref = want(s)
    assert np.array_equal(run(s), ref)
    assert np.array_equal(run(s, form="f8", split=3), ref)


@pytest.mark.parametrize("N", [16, 200])
def test_sliced_call_under_capture_and_on_other_streams(N):
    # captured calls take the tile kernels where slices would need the
    # workspace; eager calls on several streams share it in order
    F, T = 2, 4096
    x, y = rand_frame(1, T, F, N), rand_frame(2, T, F, N)
    d, e = torch.from_numpy(x).to(DEV), torch.from_numpy(y).to(DEV)
    wx, wy = want(x), want(y)
    vis = torch.zeros(vis_shape(N, F), dtype=torch.int32, device=DEV)
    with Plan(N, F, T) as p:
        p.correlate(d)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            p.correlate(d, vis)
        for src, ref in ((x, wx), (y, wy), (x, wx)):
            d.copy_(torch.from_numpy(src))
            vis.zero_()
            g.replay()
            other = p.correlate(e)
            torch.cuda.synchronize()
            assert np.array_equal(vis.cpu().numpy(), ref)
            assert np.array_equal(other.cpu().numpy(), wy)
        d.copy_(torch.from_numpy(x))
        streams = [torch.cuda.Stream() for _ in range(3)]
        outs = [torch.empty_like(vis) for _ in range(6)]
        torch.cuda.synchronize()
        for k, o in enumerate(outs):
            p.correlate(d if k % 2 else e, o, stream=streams[k % 3])
        torch.cuda.synchronize()
        for k, o in enumerate(outs):
            assert np.array_equal(o.cpu().numpy(), wx if k % 2 else wy)
        del g
