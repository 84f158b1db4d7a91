"""Beamforming launches at the edges of their workgroups: rows per workgroup
(128, 256 or 512), component tiles per launch (1..6, several launches above 192
columns), and rows at any byte alignment, against the oracle, exact."""
import numpy as np
import pytest
import torch

import oracle
from paper_1503_06202_amd import Plan

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("N,F,T,B,shift", [
    (144, 64, 1537, 33, 0), (200, 64, 1600, 64, 0),            # 512 rows, one row in the last
    (64, 64, 1537, 40, 0), (144, 3, 129, 48, 0),               # 128 rows
    (256, 2, 257, 65, 0), (130, 2, 255, 96, 0),                # five, six tiles
    (96, 1, 130, 97, 0), (48, 1, 70, 129, 0), (33, 1, 40, 193, 0),  # several launches
    (1, 1, 1, 1, 0), (15, 2, 33, 2, 0), (17, 1, 31, 17, 0), (127, 3, 129, 7, 0),
    (129, 5, 300, 20, 0), (333, 2, 513, 60, 0),
    (160, 3, 200, 9, 1), (128, 2, 129, 70, 3), (97, 2, 128, 5, 7),  # odd first address
])
def test_beam_workgroups(N, F, T, B, shift):
    rng = np.random.default_rng(N * 7 + B)
    s = rng.integers(0, 256, (T, F, N), dtype=np.uint8)
    w = rng.integers(-127, 128, (F, B, N, 2)).astype(np.int8)
    print(f"beams N={N} F={F} T={T} B={B} +{shift}", flush=True)
    # the frame ends where its allocation ends
    buf = torch.zeros(s.size + shift, dtype=torch.uint8, device=DEV)
    d = buf[shift:].view(T, F, N)
    d.copy_(torch.from_numpy(s))
    with Plan(N, F, T, beams=B) as p:
        p.set_weights(w)
        y = p.beamform(d).cpu().numpy()
    assert np.array_equal(y, oracle.beamform(s, w).astype(np.int32))
