"""Batches whose largest frames run by the packed path: those and the others
beside them, plain and replayed, against single plans' tile kernels, exact."""
import pytest
import torch

from paper_1503_06202_amd import BatchPlan, Plan, vis_shape

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")

# (N, F, T): few tiles in all (large from 1.1 M tile-samples), and many
FEW = [(64, 2, 300), (1024, 2, 16384), (1090, 1, 33000), (17, 1, 5)]
MANY = [(2048, 4, 8192), (300, 2, 1000), (1537, 4, 13001), (128, 3, 129)]


def frames(insts, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return [torch.randint(0, 256, (T, F, N), generator=g, device=DEV, dtype=torch.uint8)
            for N, F, T in insts]


def want(inst, x):
    with Plan(*inst, kernel=1) as p:
        return p.correlate(x)


@pytest.mark.parametrize("insts", [FEW, MANY, MANY[:1]])
@pytest.mark.parametrize("form,accumulate", [("i8", False), ("f8", True)])
def test_batch_with_large_frames(insts, form, accumulate):
    x = frames(insts, 5)
    ref = [want(i, a) for i, a in zip(insts, x)]
    base = 7 if accumulate else 0
    vis = [torch.full(vis_shape(N, F), 7, dtype=torch.int32, device=DEV) for N, F, T in insts]
    with BatchPlan(insts, form=form, accumulate=accumulate) as bp:
        for rep in range(4):
            print(f"batch of {len(insts)} {form} {rep}", flush=True)
            for v in vis:
                v.fill_(7)
            bp.correlate(x, vis, graph=rep > 0)
            for k, v in enumerate(vis):
                assert torch.equal(v, ref[k] + base), (k, insts[k])
        # some instances only, on another stream
        for v in vis:
            v.fill_(7)
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        active = [a if k % 2 == 0 else None for k, a in enumerate(x)]
        bp.correlate(active, vis, stream=s, graph=True)
        s.synchronize()
        for k, v in enumerate(vis):
            assert torch.equal(v, ref[k] + base if k % 2 == 0 else torch.full_like(v, 7))




# batches of few tiles whose largest frame, or all frames, run packed
FEW_PACKED = [(64, 2, 300), (1536, 2, 20000), (1090, 1, 33000), (17, 1, 5)]


@pytest.mark.parametrize("insts", [FEW_PACKED, [(2048, 2, 16384), (64, 3, 1000), (1090, 2, 20000)],
                                   [(1537, 4, 13001)]])
@pytest.mark.parametrize("form,accumulate", [("i8", False), ("f8", True)])
def test_batch_of_few_tiles(insts, form, accumulate):
    test_batch_with_large_frames(insts, form, accumulate)


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("insts", [FEW_PACKED, MANY])
def test_captured_after_a_call_by_the_packed_path(insts, graph):
    # a program's usual order: one call, then the same call captured; other
    # eager calls (the same buffers) between the replays
    x = frames(insts, 9)
    y = [a.clone() for a in x]
    ref = [want(i, a) for i, a in zip(insts, x)]
    other = frames(insts, 10)
    ref_other = [want(i, a) for i, a in zip(insts, other)]
    vis = [torch.zeros(vis_shape(N, F), dtype=torch.int32, device=DEV) for N, F, T in insts]
    print(f"captured batch of {len(insts)} graph={graph}", flush=True)
    with BatchPlan(insts) as bp:
        bp.correlate(x, vis, graph=graph)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            bp.correlate(x, vis, graph=graph)
        for src, want_now in ((y, ref), (other, ref_other), (y, ref)):
            for a, b in zip(x, src):
                a.copy_(b)
            for replayed in (True, False, True):
                for v in vis:
                    v.zero_()
                if replayed:
                    g.replay()
                else:
                    bp.correlate(x, vis, graph=graph)
                torch.cuda.synchronize()
                for k, v in enumerate(vis):
                    assert torch.equal(v, want_now[k]), (k, insts[k], replayed)
        del g
