"""No 16-byte read passes the frame's end.

The kernels read rows below ``fast_rows`` (csrc/xeng_internal.hpp) in 16-byte
pieces, the last of which reads on past a channel's inputs.  A host build of
that function is held against the addresses themselves: every piece of every
row it allows, rows of the history before the frame included, ends inside the
frame, and the next row has one that does not.  Small N is where a piece
reaches over several channels and rows.
"""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "xeng_internal.hpp"
#include <cstdio>

int main() {
  long long checked = 0;
  for (int N = 1; N <= 40; ++N)
    for (int F = 1; F <= 20; ++F)
      for (int T = 1; T <= 70; T += T < 20 ? 1 : 7)
        for (int f = 0; f < F; ++f) {
          const int fast = xeng::fast_rows(T, N, f, F);
          // the last piece of a row is the one that reaches furthest
          auto inside = [&](int t) {
            return ((long long)t * F + f) * N + (N + 15) / 16 * 16 <= (long long)T * F * N;
          };
          for (int t = -20; t < fast; ++t)
            if (!inside(t)) return std::printf("N %d F %d T %d f %d row %d\n", N, F, T, f, t), 1;
          if (fast > T) return std::printf("N %d F %d T %d f %d: %d rows\n", N, F, T, f, fast), 1;
          if (fast < T && inside(fast))
            return std::printf("N %d F %d T %d f %d: row %d left out\n", N, F, T, f, fast), 1;
          // a workgroup of several channels goes by its last one
          if (f && fast > xeng::fast_rows(T, N, f - 1, F))
            return std::printf("N %d F %d T %d f %d: more rows than f - 1\n", N, F, T, f), 1;
          ++checked;
        }
  // rows of 2^31 bytes and more
  if (xeng::fast_rows(3, 32768, 65535, 65536) != 3 || xeng::fast_rows(3, 32767, 65535, 65536) != 2 ||
      xeng::fast_rows(3, 32767, 0, 65540) != 3 || xeng::fast_rows(1 << 24, 1, 0, 1) != (1 << 24) - 15)
    return std::printf("large rows\n"), 1;
  std::printf("ok %lld\n", checked);
  return 0;
}
"""


def test_pieces_end_inside_the_frame(tmp_path):
    src, exe = tmp_path / "bounds.cpp", tmp_path / "bounds"
    src.write_text(PROGRAM)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(rocm, "include"),
                    "-I", os.path.join(ROOT, "paper_1503_06202_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True, timeout=120)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and res.stdout.startswith("ok "), res.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("N", range(1, 8))
@pytest.mark.parametrize("F,T", [(1, 64), (1, 200), (2, 128), (9, 130), (17, 64)])
def test_fewest_inputs_in_every_form(N, F, T):
    import torch

    import oracle
    from paper_1503_06202_amd import BatchPlan, Plan, vis_shape
    from paper_1503_06202_amd.engine import correlate_batch_noalloc

    dev = torch.device("cuda:0")
    print(f"N={N} F={F} T={T}", flush=True)
    rng = np.random.default_rng(100 * N + F + T)
    D = 40
    ext = rng.integers(0, 256, (D + T, F, N), dtype=np.uint8)
    s = np.ascontiguousarray(ext[D:])
    want = oracle.to_int32(oracle.correlate(s))
    dext = torch.from_numpy(ext).to(dev)
    d = dext[D:]

    def same(v, ref):
        assert np.array_equal(v.cpu().numpy(), ref)

    for form, kernel, split in (("i8", 0, 0), ("f8", 0, 2), ("i8", 1, 1), ("f8", 1, 2),
                                ("i8", 4, 0), ("i8", 5, 2)):
        with Plan(N, F, T, form=form, kernel=kernel, split_t=split) as p:
            same(p.correlate(d), want)
    vis = [torch.empty(vis_shape(N, F), dtype=torch.int32, device=dev) for _ in range(2)]
    with BatchPlan([(N, F, T)] * 2, split_t=[1, 2]) as bp:
        bp.correlate([d, d], vis)
        for v in vis:
            same(v, want)
    correlate_batch_noalloc([(N, F, T)], [d], vis[:1])
    same(vis[0], want)
    gate = (np.arange(T) // 30 % 3).astype(np.int32)
    with Plan(N, F, T, gates=3) as p:
        same(p.correlate_gated(d, gate, 3), oracle.to_int32(oracle.correlate_gated(s, gate, 3)))
    delays = np.full(N, 33, np.int32)
    with Plan(N, F, T) as p:
        p.set_delays(delays, D)
        same(p.correlate(d), oracle.to_int32(oracle.correlate_shifted(ext, D, delays)))
    words = rng.integers(0, 1 << N, (T, F, 1), dtype=np.uint32)
    words[rng.random((T, F, 1)) < 0.9] = 0
    own = d.clone()
    with Plan(N, F, T, flagged=True) as p:
        v, c = p.correlate_flagged(own, torch.from_numpy(words.view(np.int32)).to(dev))
    rv, rc = oracle.correlate_flagged(s, words)
    same(v, oracle.to_int32(rv))
    assert np.array_equal(c.cpu().numpy().astype(np.int64), rc)
    w = rng.integers(-127, 128, (F, 3, N, 2)).astype(np.int8)
    with Plan(N, F, T, beams=3) as p:
        p.set_weights(w)
        same(p.beamform(d), oracle.beamform(s, w).astype(np.int32))
