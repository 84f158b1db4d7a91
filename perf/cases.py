"""Workloads of the X-engine: what a program that uses it calls, over the range it calls it.

Every case is one pass through a public entry point (``Plan``, ``BatchPlan``,
``correlate_batch_noalloc``) on device buffers that the program holds: samples
uint8 ``[T][F][N]`` (4+4-bit offset-binary complex), int32 visibilities, and
the plan made once for the shape.  Inputs are drawn on the GPU from the seed
alone: sky-noise Gaussians that are about 50% correlated between inputs
(2.5 x N(0, 1) codes, mild clipping), one channel in twenty with a strong
tone, as in the repository's synthetic frames.

Kinds of case (field ``kind``):

* ``plain``    N, F, T, form ("i8" / "f8"), accumulate: one frame's correlation;
* ``gated``    + gates, period: samples folded into phase bins;
* ``shifted``  + dmax, pattern ("groups": a delay per 16 inputs, "stations":
  half the array delayed): integer delays with history before the frame;
* ``flagged``  + recipe ("rare" / "heavy"): invalid samples excluded, pair
  counts, renormalised output;
* ``beams``    + beams: phased beams at the sample cadence;
* ``batch``    count, mix, F, tmax, odd, mode ("launch", "graph", "noalloc"):
  many uneven frames in one launch.
"""
import math
import random

import numpy as np
import torch

from paper_1503_06202_amd.engine import BatchPlan, Plan, correlate_batch_noalloc, vis_shape

DEV = "cuda:0"


def listed():
    return [
        # the smallest call: a bench-top array of 16 inputs, one channel, a short dump
        dict(name="tiny", kind="plain", N=16, F=1, T=256, form="i8", accumulate=False),
        # an ordinary small frame: a 64-input station, as in the batched mix, called alone
        dict(name="station", kind="plain", N=64, F=4, T=8192, form="i8", accumulate=False),
        # the Pathfinder's 256 inputs, a node's channels, one 84 ms frame
        dict(name="pathfinder", kind="plain", N=256, F=64, T=32768, form="i8", accumulate=False),
        # an array whose inputs and frame length fit no tile, integrating on
        dict(name="ragged", kind="plain", N=1090, F=8, T=20011, form="i8", accumulate=True),
        # the headline: the full array's 2048 inputs, 16 channels
        dict(name="full_array", kind="plain", N=2048, F=16, T=32768, form="i8", accumulate=False),
        # one frame of the streaming loop in the FP8 form, added to its integration
        dict(name="stream_f8", kind="plain", N=2048, F=4, T=32768, form="f8", accumulate=True),
        # a pulsar folded into 16 phase bins on one stream frame
        dict(name="gated", kind="gated", N=2048, F=4, T=32768, gates=16, period=8192),
        # inputs spread over many cable lengths and sites: a delay for every 16 of them
        dict(name="shifted", kind="shifted", N=2048, F=16, T=32768, dmax=60000, pattern="groups"),
        # a healthy array's rare faults: lost packets, saturated inputs, overflows
        dict(name="flagged", kind="flagged", N=2048, F=16, T=32768, recipe="rare"),
        # a few tracking beams of the full array
        dict(name="beams16", kind="beams", N=2048, F=16, T=32768, beams=16),
        # many beams of the full array
        dict(name="beams64", kind="beams", N=2048, F=16, T=32768, beams=64),
        # 48 uneven frames (N 64..2048, T 8192..32768) replayed as one graph
        dict(name="batch48", kind="batch", count=48, mix=5, F=4, tmax=32768, odd=False,
             mode="graph"),
    ]


# ---------------------------------------------------------------------------
# drawn cases


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo_n, hi_n, ragged, most_bytes=1 << 29, most_cmac=3e11):
    """N, F, T with sizes spread over their logarithms, within a frame's cost."""
    while True:
        N = _log(rng, lo_n, hi_n)
        if not ragged:
            N = max(16, (N + 8) // 16 * 16)
        F = _log(rng, 1, 64)
        T = _log(rng, 128, 65536)
        if not ragged:
            T = max(128, T // 64 * 64)
        if T * F * N <= most_bytes and T * F * N * (N + 1) / 2 <= most_cmac:
            return N, F, T


def draw(rng):
    kind = rng.choice(["plain"] * 6 + ["gated", "shifted", "flagged", "beams", "beams", "batch"])
    ragged = rng.random() < 0.5
    if kind == "plain":
        N, F, T = _size(rng, 8, 2048, ragged)
        return dict(kind=kind, N=N, F=F, T=T, form=rng.choice(["i8", "i8", "f8"]),
                    accumulate=rng.random() < 0.4)
    if kind == "gated":
        N, F, T = _size(rng, 16, 1024, ragged)
        return dict(kind=kind, N=N, F=F, T=T, gates=rng.choice([2, 3, 8, 16]),
                    period=_log(rng, 256, 16384))
    if kind == "shifted":
        N, F, T = _size(rng, 32, 2048, ragged)
        while T > 32768:
            T //= 2
        dmax = min(_log(rng, 64, 16384), (1 << 30) // (F * N))
        return dict(kind=kind, N=N, F=F, T=T, dmax=dmax,
                    pattern=rng.choice(["groups", "groups", "stations"]))
    if kind == "flagged":
        N, F, T = _size(rng, 16, 2048, ragged)
        return dict(kind=kind, N=N, F=F, T=T, recipe=rng.choice(["rare", "rare", "heavy"]))
    if kind == "beams":
        N, F, T = _size(rng, 32, 2048, ragged, most_bytes=1 << 28)
        return dict(kind=kind, N=N, F=F, T=T, beams=_log(rng, 1, 96))
    return dict(kind=kind, count=rng.randint(2, 24), mix=rng.randrange(1 << 20), F=rng.randint(1, 4),
                tmax=rng.choice([2048, 8192, 16384]), odd=ragged,
                mode=rng.choice(["launch", "graph", "graph", "noalloc"]))


def _instances(case):
    """(N, F, T) of a batch, from its own mix number (not from the inputs' seed)."""
    r = random.Random(case["mix"])
    out = []
    for _ in range(case["count"]):
        N = r.choice([64, 128, 256, 512, 1024, 2048])
        T = case["tmax"] // r.choice([1, 2, 4])
        if case["odd"]:
            N, T = N - r.randint(0, N // 3), T - r.randint(0, T // 3)
        out.append((N, case["F"], T))
    return out


# ---------------------------------------------------------------------------
# inputs


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _samples(g, N, F, T):
    """A frame uint8 [T][F][N]: correlated sky noise, every 20th channel (one at least) toned."""
    out = torch.empty((T, F, N), dtype=torch.uint8, device=DEV)
    gain = torch.rand((N, 1), generator=g, device=DEV) + 0.5
    phase = torch.rand((N,), generator=g, device=DEV) * (2 * math.pi)
    tone = torch.randint(0, F, (1 + F // 20,), generator=g, device=DEV)
    toned = torch.zeros((F,), device=DEV).index_fill_(0, tone, 6.0)
    step = max(1, min(T, (1 << 26) // (F * N)))
    for t0 in range(0, T, step):
        n = min(step, T - t0)
        x = torch.randn((n, F, N, 2), generator=g, device=DEV)
        x += torch.randn((n, F, 1, 2), generator=g, device=DEV) * gain
        x *= 2.5
        t = torch.arange(t0, t0 + n, device=DEV, dtype=torch.float32)
        ang = (t * (2 * math.pi * 0.1375)).remainder(2 * math.pi)[:, None] + phase
        x[..., 0] += toned[:, None] * torch.cos(ang)[:, None, :]
        x[..., 1] += toned[:, None] * torch.sin(ang)[:, None, :]
        u = x.round_().clamp_(-8, 7).add_(8).to(torch.uint8)
        out[t0:t0 + n] = u[..., 0] * 16 + u[..., 1]
        del x, u, ang
    return out


def _delays(case, seed):
    N, D = case["N"], case["dmax"]
    if case["pattern"] == "stations":
        n = np.arange(N)
        return np.where(n < (N // 2) // 128 * 128, 0, (2 * D) // 3).astype(np.int32)
    r = np.random.default_rng(seed)
    return np.repeat(r.integers(0, D + 1, (N + 15) // 16), 16)[:N].astype(np.int32)


def _flags(g, case):
    """Boolean [T][F][N]: lost packets (16 samples x 8 channels, all inputs),
    saturated inputs (64 samples, all channels) and single overflows."""
    N, F, T = case["N"], case["F"], case["T"]
    packet, sat, over = (1e-3, 1e-3, 1e-5) if case["recipe"] == "rare" else (5e-2, 2e-2, 1e-4)
    rand = lambda *s: torch.rand(s, generator=g, device=DEV)  # noqa: E731
    m = rand(-(-T // 64), N) < sat
    m = m.repeat_interleave(64, 0)[:T][:, None, :].expand(T, F, N).contiguous()
    p = rand(-(-T // 16), -(-F // 8)) < packet
    m |= p.repeat_interleave(16, 0)[:T].repeat_interleave(8, 1)[:, :F][:, :, None]
    k = max(1, int(T * F * N * over))
    m.view(-1)[torch.randint(0, T * F * N, (k,), generator=g, device=DEV)] = True
    return m


def _pack(mask):
    """Flag words int32 [T][F][ceil(N/32)], bit i % 32 of word i // 32 = input i invalid."""
    T, F, N = mask.shape
    W = (N + 31) // 32
    out = torch.empty((T, F, W), dtype=torch.int32, device=mask.device)
    bit = torch.arange(32, device=mask.device)
    step = max(1, (1 << 24) // (F * W * 32))
    for t0 in range(0, T, step):
        m = torch.zeros((min(step, T - t0), F, W * 32), dtype=torch.int64, device=mask.device)
        m[..., :N] = mask[t0:t0 + step]
        w = (m.view(-1, F, W, 32) << bit).sum(-1)
        out[t0:t0 + step] = torch.where(w >= 1 << 31, w - (1 << 32), w).to(torch.int32)
    return out


def _weights(case, seed):
    """Phase weights 127 e^{-i phi} of a line of inputs, int8 [F][B][N][2]."""
    N, F, B = case["N"], case["F"], case["beams"]
    r = np.random.default_rng(seed)
    s, cal = r.uniform(-0.9, 0.9, B), r.uniform(0, 2 * np.pi, N)
    nu = 400e6 + 400e6 * (np.arange(F) + 0.5) / F
    phi = (2 * np.pi / 2.998e8) * nu[:, None, None] * s[:, None] * (0.3 * np.arange(N)) + cal
    return np.rint(127 * np.stack([np.cos(phi), -np.sin(phi)], -1)).astype(np.int8)


def _gate(case):
    t = np.arange(case["T"], dtype=np.int64)
    return ((t % case["period"]) * case["gates"] // case["period"]).astype(np.int32)


def _inputs(case, seed):
    """Everything drawn from the seed; prepare() and exact() share it."""
    g = _gen(seed)
    kind = case["kind"]
    if kind == "batch":
        return {"frames": [_samples(g, *i) for i in _instances(case)]}
    N, F, T = case["N"], case["F"], case["T"]
    if kind == "shifted":
        return {"ext": _samples(g, N, F, T + case["dmax"]), "delays": _delays(case, seed)}
    got = {"samples": _samples(g, N, F, T)}
    if kind == "flagged":
        got["mask"] = _flags(g, case)
    if kind == "plain" and case["accumulate"]:
        # the integration so far
        got["vis"] = torch.randint(-1000, 1000, vis_shape(N, F), generator=g, device=DEV,
                                   dtype=torch.int32)
        i = torch.arange(N, device=DEV)
        got["vis"][:, i * N - i * (i - 1) // 2, 1] = 0
    if kind == "beams":
        got["weights"] = _weights(case, seed)
    return got


def prepare(case, seed):
    s = dict(_inputs(case, seed), case=case)
    kind = case["kind"]
    if kind == "batch":
        inst = _instances(case)
        s["inst"] = inst
        s["vis"] = [torch.empty(vis_shape(N, F), dtype=torch.int32, device=DEV) for N, F, T in inst]
        if case["mode"] != "noalloc":
            s["plan"] = BatchPlan(inst)
        return s
    N, F, T = case["N"], case["F"], case["T"]
    if "vis" not in s and kind != "beams":
        lead = (case["gates"],) if kind == "gated" else ()
        s["vis"] = torch.empty(lead + vis_shape(N, F), dtype=torch.int32, device=DEV)
    if kind == "plain":
        s["plan"] = Plan(N, F, T, form=case["form"], accumulate=case["accumulate"])
    elif kind == "gated":
        s["gate"] = _gate(case)
        s["plan"] = Plan(N, F, T, gates=case["gates"])
    elif kind == "shifted":
        s["samples"] = s["ext"][case["dmax"]:]
        s["plan"] = Plan(N, F, T)
        s["plan"].set_delays(s["delays"], case["dmax"])
    elif kind == "flagged":
        s["flags"] = _pack(s.pop("mask"))
        B = N * (N + 1) // 2
        s["counts"] = torch.empty((F, B), dtype=torch.int32, device=DEV)
        s["norm"] = torch.empty(vis_shape(N, F), dtype=torch.float32, device=DEV)
        s["plan"] = Plan(N, F, T, flagged=True)
    else:
        s["out"] = torch.empty((T, F, case["beams"], 2), dtype=torch.int32, device=DEV)
        s["plan"] = Plan(N, F, T, beams=case["beams"])
        s["plan"].set_weights(s.pop("weights"))
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "plain" or kind == "shifted":
        return s["plan"].correlate(s["samples"], s["vis"])
    if kind == "gated":
        return s["plan"].correlate_gated(s["samples"], s["gate"], case["gates"], s["vis"])
    if kind == "flagged":
        vis, counts = s["plan"].correlate_flagged(s["samples"], s["flags"], s["vis"], s["counts"])
        norm = s["plan"].normalize(vis, counts, float(case["T"]), s["norm"])
        return {"vis": vis, "counts": counts, "norm": norm, "samples": s["samples"]}
    if kind == "beams":
        return s["plan"].beamform(s["samples"], s["out"])
    if case["mode"] == "noalloc":
        correlate_batch_noalloc(s["inst"], s["frames"], s["vis"])
    else:
        s["plan"].correlate(s["frames"], s["vis"], graph=case["mode"] == "graph")
    return s["vis"]


def work(case):
    """Complex MACs as 8 operations; samples (and flags) read once, results written once."""
    if case["kind"] == "batch":
        each = [work(dict(kind="plain", N=N, F=F, T=T, accumulate=False))
                for N, F, T in _instances(case)]
        return {k: sum(w[k] for w in each) for k in ("bytes", "flops")}
    N, F, T, kind = case["N"], case["F"], case["T"], case["kind"]
    B = N * (N + 1) // 2
    if kind == "beams":
        b = case["beams"]
        return {"bytes": T * F * N + 8 * T * F * b + 2 * F * b * N, "flops": 8 * T * F * b * N}
    nbytes, flops = T * F * N + 8 * F * B, 8 * T * F * B
    if kind == "plain" and case["accumulate"]:
        nbytes += 8 * F * B
    if kind == "gated":
        nbytes += 8 * F * B * (case["gates"] - 1)
    if kind == "flagged":
        # flags; counts and the renormalised output beside the visibilities, which are read again
        nbytes += T * F * ((N + 31) // 32) * 4 + (4 + 4 + 8 + 8) * F * B
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------------------
# the same in 64 bits, with torch alone


def _parts(x):
    """Real and imaginary parts of samples, float64."""
    return (x >> 4).double().sub_(8), (x & 15).double().sub_(8)


def _triangle(N):
    return torch.triu_indices(N, N, device=DEV)


def _gram(x, tri):
    """[B][2] int64: sum_t x_i conj(x_j) of samples x [T][N], i <= j (exact below 2^53)."""
    N = x.shape[1]
    re = torch.zeros((N, N), dtype=torch.float64, device=DEV)
    mr = torch.zeros((N, N), dtype=torch.float64, device=DEV)
    for t0 in range(0, x.shape[0], 32768):
        r, m = _parts(x[t0:t0 + 32768])
        rt, mt = r.t().contiguous(), m.t().contiguous()
        re += rt @ r
        re += mt @ m
        mr += mt @ r
    im = mr - mr.t()
    return torch.stack([re[tri[0], tri[1]], im[tri[0], tri[1]]], -1).to(torch.int64)


def exact(case, seed):
    inp = _inputs(case, seed)
    kind = case["kind"]
    if kind == "batch":
        got = []
        for x in inp["frames"]:
            tri = _triangle(x.shape[2])
            got.append(torch.stack([_gram(x[:, f], tri) for f in range(x.shape[1])]))
        return got
    N, F, T = case["N"], case["F"], case["T"]
    if kind == "beams":
        w = torch.from_numpy(inp["weights"]).to(DEV).double()
        out = torch.empty((T, F, case["beams"], 2), dtype=torch.int64, device=DEV)
        for f in range(F):
            r, m = _parts(inp["samples"][:, f])
            wr, wi = w[f, :, :, 0].t().contiguous(), w[f, :, :, 1].t().contiguous()
            out[:, f, :, 0] = (r @ wr - m @ wi).to(torch.int64)
            out[:, f, :, 1] = (r @ wi + m @ wr).to(torch.int64)
        return out
    tri = _triangle(N)
    if kind == "shifted":
        x = torch.empty((T, F, N), dtype=torch.uint8, device=DEV)
        for n0 in range(0, N, 16):
            t0 = case["dmax"] - int(inp["delays"][n0])
            x[:, :, n0:n0 + 16] = inp["ext"][t0:t0 + T, :, n0:n0 + 16]
    else:
        x = inp["samples"]
    if kind == "gated":
        gate = torch.from_numpy(_gate(case)).to(DEV)
        return torch.stack([torch.stack([_gram(x[:, f][gate == g], tri) for f in range(F)])
                            for g in range(case["gates"])])
    if kind != "flagged":
        vis = torch.stack([_gram(x[:, f], tri) for f in range(F)])
        return vis + inp["vis"] if "vis" in inp else vis
    x = torch.where(inp["mask"], torch.tensor(0x88, dtype=torch.uint8, device=DEV), x)
    vis = torch.stack([_gram(x[:, f], tri) for f in range(F)])
    counts = []
    for f in range(F):
        ok = (~inp["mask"][:, f]).double()
        counts.append((ok.t().contiguous() @ ok)[tri[0], tri[1]].to(torch.int64))
    counts = torch.stack(counts)
    c = counts.double()[..., None]
    norm = torch.where(c > 0, vis.double() * float(T) / c.clamp(min=1), torch.zeros_like(c))
    return {"vis": vis, "counts": counts, "norm": norm, "samples": x}
