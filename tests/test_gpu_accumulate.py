"""Accumulating writes of every kernel family: the frame's sums land on every
baseline of a vis that already holds numbers, and the rest of its memory stays."""
import numpy as np
import pytest
import torch

import oracle
from paper_1503_06202_amd import Plan, vis_shape

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("form", ["i8", "f8"])
@pytest.mark.parametrize("N,F,T,kernel", [
    (129, 2, 130, 1), (300, 3, 100, 0), (257, 1, 64, 1), (127, 2, 65, 1),   # tiles
    (200, 2, 130, 0), (256, 1, 4000, 0),                                    # channel kernel
    (64, 3, 200, 0), (17, 5, 65, 0),                                        # small arrays
    (1025, 1, 5300, 0), (657, 2, 14000, 0), (1281, 2, 2600, 0),             # packed
])
def test_accumulate_into_vis(N, F, T, kernel, form):
    rng = np.random.default_rng(N + T)
    s = rng.integers(0, 256, (T, F, N), dtype=np.uint8)
    print(f"accumulate N={N} F={F} T={T} {form}", flush=True)
    n = int(np.prod(vis_shape(N, F)))
    buf = torch.randint(-9999, 9999, (n + 256,), device=DEV, dtype=torch.int32)
    before = buf.clone()
    vis = buf[128:128 + n].view(vis_shape(N, F))
    with Plan(N, F, T, form=form, accumulate=True, kernel=kernel) as p:
        p.correlate(torch.from_numpy(s).to(DEV), vis)
        torch.cuda.synchronize()
    got = (buf - before).cpu().numpy()
    assert not got[:128].any() and not got[128 + n:].any()
    ref = oracle.to_int32(oracle.correlate(s)).reshape(-1)
    assert np.array_equal(got[128:128 + n], ref)
