"""Frames whose rows are not 16-byte aligned, through the vector loads, against
the CPU oracle, bit-exact.

Whole chunks of 64 samples are read in 16-byte pieces at any alignment; the
last piece of a row reads on into the next channel or row, except in the
frame's very last row.  The shapes put that row into a whole chunk (T a
multiple of 64), into a ragged one, and before it, in the first, the last and
the only channel, for every kernel that reads frames: the tile kernel (int8
and FP8, sliced and not), the channel kernel, the gated, batched and shifted
forms.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1503_06202_amd import BatchPlan, Plan, vis_shape
from paper_1503_06202_amd.engine import correlate_batch_noalloc

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def rand_frame(seed, T, F, N):
    return np.random.default_rng(seed).integers(0, 256, (T, F, N), dtype=np.uint8)


def want(s):
    return oracle.to_int32(oracle.correlate(s))


def at_offset(s, offset):
    """The frame on the GPU, `offset` bytes into an allocation that it fills to its end."""
    raw = torch.empty(offset + s.size, dtype=torch.uint8, device=DEV)
    view = raw[offset:].view(s.shape)
    view.copy_(torch.from_numpy(s))
    return view


@pytest.mark.parametrize("offset", [0, 5])
@pytest.mark.parametrize("F", [1, 3])
@pytest.mark.parametrize("N,T", [(1, 64), (7, 128), (17, 192), (100, 256), (127, 320), (129, 256),
                                 (145, 640), (250, 576), (255, 321), (257, 257), (500, 192)])
def test_ragged_rows(N, T, F, offset):
    s = rand_frame(N * T + F, T, F, N)
    d, ref = at_offset(s, offset), want(s)
    for form, kernel, split in (("i8", 0, 0), ("i8", 1, 1), ("i8", 1, 2), ("f8", 1, 0), ("i8", 5, 2)):
        with Plan(N, F, T, form=form, kernel=kernel, split_t=split) as p:
            got = p.correlate(d)
            torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy(), ref), (form, kernel, split)


@pytest.mark.parametrize("N,T", [(33, 256), (200, 320), (301, 448)])
def test_ragged_forms(N, T):
    F, D = 2, 70
    ext = rand_frame(N, D + T, F, N)
    s = np.ascontiguousarray(ext[D:])
    ref = want(s)
    dev = at_offset(ext, 3)
    frame = dev[D:]
    vis = [torch.empty(vis_shape(N, F), dtype=torch.int32, device=DEV) for _ in range(2)]
    for split in (1, 3):
        with BatchPlan([(N, F, T)] * 2, split_t=[split] * 2) as bp:
            bp.correlate([frame, frame], vis)
            torch.cuda.synchronize()
            assert all(np.array_equal(v.cpu().numpy(), ref) for v in vis), split
    correlate_batch_noalloc([(N, F, T)], [frame], vis[:1])
    torch.cuda.synchronize()
    assert np.array_equal(vis[0].cpu().numpy(), ref)
    gate = (np.arange(T) // 50 % 3).astype(np.int32)
    with Plan(N, F, T, gates=3) as p:
        got = p.correlate_gated(frame, gate, 3).cpu().numpy()
    assert np.array_equal(got, oracle.to_int32(oracle.correlate_gated(s, gate, 3)))
    blocks = np.repeat([0, 70, 33], 128)[:N].astype(np.int32)
    with Plan(N, F, T) as p:
        p.set_delays(blocks, D)
        got = p.correlate(frame).cpu().numpy()
    assert np.array_equal(got, oracle.to_int32(oracle.correlate_shifted(ext, D, blocks)))
    flags = (np.random.default_rng(N).random((T, F, N)) < 0.01)
    words = np.packbits(np.pad(flags, ((0, 0), (0, 0), (0, -N % 32))), axis=-1, bitorder="little")
    fl = torch.from_numpy(np.ascontiguousarray(words).view(np.int32).reshape(T, F, -1)).to(DEV)
    with Plan(N, F, T, flagged=True) as p:
        v, c = p.correlate_flagged(frame, fl)
        torch.cuda.synchronize()
    rv, rc = oracle.correlate_flagged(s, words.view(np.uint32).reshape(T, F, -1))
    assert np.array_equal(v.cpu().numpy(), oracle.to_int32(rv))
    assert np.array_equal(c.cpu().numpy().astype(np.int64), rc)
