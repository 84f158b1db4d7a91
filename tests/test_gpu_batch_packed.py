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


