"""The work that is measured: what a user of this package has it do at a denoising step.

A video DiT that schedules its frames asynchronously spends its attention in five kinds of call, and the
cases here are those calls at the repository's own workloads (`paper_2606_06309_amd/workloads.py`) and at
generic clips around them:

  step     a skipped step: project the latents, attend with the keyframes' queries, scatter the rows back
  attend   attention alone; with every frame a keyframe it is a warm-up step or a Rhythmic Point
  mask     attention of the keyframes over the keyframes only (the "w/o projection" ablation)
  cache    the rolling cache of one layer: initialise, shift and store, project into the keys and values
  select   cosine similarity of a video's frames, the input of the content-aware keyframe choice
  project  the latents of a batch projected to a step in between

Sizes: T frames of H x W tokens, `heads` heads of `dim`, M keyframes spread evenly over the frames. Latents
have C channels on an Hl x Wl grid.
"""
import math

import torch

from paper_2606_06309_amd import binding as rf

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
TIMES = (24.0, 21.0, 23.0)            # snapshots at 24 and 21, the step in between at 23
T_WARM, T_RHYTHMIC, T_SKIP = 42.0, 39.0, 40.0


def _frames(T, M):
    """M frames spread evenly over T with both ends among them (the first alone for M = 1)."""
    return [0] if M == 1 else [(2 * i * (T - 1) + M - 1) // (2 * (M - 1)) for i in range(M)]


def listed():
    return [
        # the smallest workload of the tests, in fp32 from end to end: latency and launches
        dict(name="step-tiny-f32", kind="step", dtype="f32", T=5, H=8, W=8, heads=2, dim=64, M=3,
             C=4, Hl=16, Wl=16),
        # a short clip at a ragged size (527 tokens a frame, five heads): nothing divides a tile
        dict(name="step-clip", kind="step", dtype="bf16", T=9, H=17, W=31, heads=5, dim=64, M=3,
             C=16, Hl=34, Wl=62),
        # the small workload: attention of a short 480p clip, every third frame a keyframe
        dict(name="attend-small", kind="attend", dtype="bf16", T=13, H=30, W=52, heads=12, dim=128, M=5),
        # the same clip in fp32, as when a bf16 pipeline is checked against full precision
        dict(name="attend-small-f32", kind="attend", dtype="f32", T=13, H=30, W=52, heads=12, dim=128, M=5),
        # a skipped step of a 480p video
        dict(name="step-480p", kind="step", dtype="bf16", T=21, H=30, W=52, heads=12, dim=128, M=6,
             C=16, Hl=60, Wl=104),
        # a warm-up step or Rhythmic Point of that video: every frame's queries over every frame
        dict(name="attend-480p-all", kind="attend", dtype="bf16", T=21, H=30, W=52, heads=12, dim=128, M=21),
        # a skipped step of that video without projected frames: keyframes over keyframes
        dict(name="mask-480p", kind="mask", dtype="bf16", T=21, H=30, W=52, heads=12, dim=128, M=6),
        # the rolling cache of one layer of that video
        dict(name="cache-480p", kind="cache", dtype="bf16", T=21, H=30, W=52, heads=12, dim=128, M=6),
        # the paper's two models at their own sizes, four keyframes
        dict(name="step-wan-1.3b", kind="step", dtype="bf16", T=21, H=45, W=80, heads=12, dim=128, M=4,
             C=16, Hl=90, Wl=160),
        dict(name="attend-cogvideox", kind="attend", dtype="bf16", T=11, H=48, W=85, heads=48, dim=64, M=4),
        # the long video, the workload of the benchmark, and the choice of its keyframes
        dict(name="step-long", kind="step", dtype="bf16", T=33, H=45, W=80, heads=24, dim=128, M=8,
             C=16, Hl=90, Wl=160),
        dict(name="select-long", kind="select", dtype="f32", B=1, C=16, T=33, H=90, W=160),
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, even over its logarithm."""
    return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    """One more case: clips of 5 to 33 frames, latent grids from 8 x 8 to 90 x 160, odd sizes as often as even
    ones. Attention stays below 8 TFLOP in bf16 and 0.5 TFLOP in fp32, data below 1 GB."""
    while True:
        kind = rng.choice(["step", "step", "attend", "attend", "mask", "cache", "select", "project"])
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        T = _log(rng, 5, 33)
        H = _log(rng, 8, 48)
        W = max(8, min(96, round(H * rng.uniform(0.6, 1.9))))
        heads, dim = _log(rng, 2, 48), rng.choice([64, 128, 128])
        M = rng.choice([2, 3, 4, max(2, T // 6), max(2, T // 4), max(2, T // 3), T])
        C = rng.choice([4, 16, 16])
        if kind in ("select", "project"):
            case = dict(kind=kind, dtype=rng.choice(["f32", "f32", "bf16"]), B=rng.choice([1, 1, 2, 5]), C=C,
                        T=T, H=2 * H if rng.random() < 0.7 else 2 * H + 1, W=2 * W + rng.choice([0, 0, 1]))
            if kind == "project":
                case["M"] = M if M < T else 2
            if case["B"] * C * T * case["H"] * case["W"] * 4 > 5e8:
                continue
            return case
        case = dict(kind=kind, dtype=dtype, T=T, H=H, W=W, heads=heads, dim=dim, M=M)
        if kind in ("mask", "cache") and M == T:
            case["M"] = M = max(2, T // 3)
        if kind == "step":
            case.update(C=C, Hl=2 * H, Wl=2 * W)
        w = work(case)
        if w["flops"] > (5e11 if dtype == "f32" else 8e12) or w["bytes"] > 1e9:
            continue
        return case


def _draws(case, seed):
    """The tensors of a case, in a fixed order from one generator: unit normals, the scale that normalised
    queries, keys and latents have."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt = DTYPES[case["dtype"]]

    def normal(*shape, dtype=dt):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).to(dtype)

    kind, T = case["kind"], case["T"]
    if kind == "select":
        # scenes of about seven frames: a shared picture and noise of each frame's own
        x = 0.3 * normal(case["B"], case["C"], T, case["H"], case["W"], dtype=torch.float32)
        for first in range(0, T, 7):
            x[:, :, first:first + 7] += normal(case["B"], case["C"], 1, case["H"], case["W"], dtype=torch.float32)
        return {"latents": x.to(dt)}
    if kind == "project":
        return {"latents": normal(case["B"], 2, case["C"], T, case["H"], case["W"])}
    S, N, heads, dim = T * case["H"] * case["W"], case["H"] * case["W"], case["heads"], case["dim"]
    t = {}
    if kind == "cache":
        for name in ("h0", "h1", "k", "v"):
            t[name] = normal(S, heads, dim)
        return t
    for name in ("q", "k", "v"):
        t[name] = normal(S, heads, dim)
    if kind == "step":
        t["latents"] = normal(1, 2, case["C"], T, case["Hl"], case["Wl"], dtype=torch.float32)
        t["full"] = normal(S, heads, dim)      # the layer's output of the step before
    return t


def prepare(case, seed):
    st = dict(case=case, **_draws(case, seed))
    kind, T = case["kind"], case["T"]
    if kind == "select":
        n = rf.rf_frame_similarity_workspace(case["B"], case["C"], T, case["H"], case["W"])
        st["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda")
        st["out"] = torch.empty((case["B"], T, T), dtype=torch.float64, device="cuda")
        return st
    st["ids"], st["mask"] = rf.rf_select_keyframes(_frames(T, case["M"]), T)
    if kind == "project":
        x = st["latents"]
        st["projected"] = torch.empty((x.shape[0],) + tuple(x.shape[2:]), dtype=x.dtype, device="cuda")
        return st
    H, W, heads, dim = case["H"], case["W"], case["heads"], case["dim"]
    if kind == "cache":
        st["others"] = [f for f in range(T) if not st["mask"][f]]
        n = rf.rf_cache_store_bytes(len(st["others"]), H * W, heads * dim, st["k"].dtype)
        st["store"] = torch.empty(n // st["k"].element_size(), dtype=st["k"].dtype, device="cuda")
        st["cache"] = rf.rf_rolling_cache()
        return st
    M = len(st["ids"])
    st["out"] = torch.empty((M * H * W, heads, dim), dtype=st["q"].dtype, device="cuda")
    n = rf.rf_attention_workspace(M, M if kind == "mask" else T, T, H, W, heads, dim, st["q"].dtype)
    st["ws"] = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
    if kind == "step":
        x = st["latents"]
        st["projected"] = torch.empty((1,) + tuple(x.shape[2:]), dtype=x.dtype, device="cuda")
    return st


def run(st):
    case, kind = st["case"], st["case"]["kind"]
    T, H, W = case["T"], case["H"], case["W"]
    if kind == "select":
        return rf.rf_frame_similarity(st["latents"], out=st["out"], workspace=st["ws"])
    if kind == "project":
        return rf.rf_project_latents(st["latents"], TIMES, st["mask"], out=st["projected"])
    if kind == "cache":
        hidden = case["heads"] * case["dim"]
        cache, store = st["cache"], st["store"]
        rf.rf_cache_init(st["others"], T, H * W, hidden, store.dtype, T_WARM, store=store, h_full=st["h0"],
                         cache=cache)
        rf.rf_cache_shift_store(cache, T_RHYTHMIC, store=store, h_full=st["h1"])
        rf.rf_cache_project_kv(cache, store, st["k"], st["v"], T_SKIP)
        return store, st["k"], st["v"]
    if kind == "mask":
        return rf.rf_frame_attention(st["q"], st["k"], st["v"], st["ids"], st["ids"], T, H, W, out=st["out"],
                                     workspace=st["ws"])
    if kind == "attend":
        return rf.rf_keyframe_attention_ws(st["q"], st["k"], st["v"], st["ids"], T, H, W, out=st["out"],
                                           workspace=st["ws"])
    projected = rf.rf_project_latents(st["latents"], TIMES, st["mask"], out=st["projected"])
    out = rf.rf_keyframe_attention_ws(st["q"], st["k"], st["v"], st["ids"], T, H, W, out=st["out"],
                                      workspace=st["ws"])
    full = rf.rf_scatter_frames(out, st["full"], st["ids"], T, H * W)
    return projected, out, full


def work(case):
    kind, T = case["kind"], case["T"]
    size = 2 if case["dtype"] == "bf16" else 4
    if kind == "select":
        n = case["C"] * case["H"] * case["W"]
        return {"bytes": case["B"] * (T * n * size + T * T * 8), "flops": case["B"] * T * (T + 1) * n}
    if kind == "project":
        n = case["B"] * case["C"] * case["H"] * case["W"]
        M = case["M"]
        return {"bytes": n * size * (3 * (T - M) + 2 * M), "flops": 3 * n * (T - M)}
    N, row, M = case["H"] * case["W"], case["heads"] * case["dim"], case["M"]
    if kind == "cache":
        # each cached frame: two states read and stored, a key and a value written
        n = (T - M) * N * row
        return {"bytes": 6 * n * size, "flops": 3 * n}
    keys = (M if kind == "mask" else T) * N
    flops = 4 * M * N * keys * row
    nbytes = (2 * M * N + 2 * keys) * row * size
    if kind == "step":
        n = case["C"] * case["Hl"] * case["Wl"]
        nbytes += n * 4 * (3 * (T - M) + 2 * M) + 2 * M * N * row * size
        flops += 3 * n * (T - M)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # four times the distance from exact() that was measured
    if case["kind"] == "select":
        return {"rel": 1e-13}                 # sums in 64 bits: 1.1e-14 over 230,400 elements
    if case["kind"] in ("cache", "project"):
        # one rounding of a blend: 1.2e-3 in bf16, 5e-8 in fp32
        return {"rel": 5e-3, "max": 1e-2} if case["dtype"] == "bf16" else {"rel": 2e-7, "max": 2e-6}
    if case["dtype"] == "bf16":
        return {"rel": 1e-2, "max": 0.1}      # outputs and probabilities rounded to bf16: 2.4e-3
    return {"rel": 1.3e-5, "max": 2e-4}       # sums in 32 bits: 3.3e-6 over 20,280 keys


def _attention(q, k, v, rows, keys):
    """softmax(q k^T / sqrt(d)) v of the listed tokens over the listed tokens, a head at a time in 64 bits."""
    heads, dim = q.shape[1], q.shape[2]
    out = torch.empty((len(rows), heads, dim), dtype=torch.float64, device=q.device)
    step = max(1, 100_000_000 // len(keys))
    for h in range(heads):
        kt = k[keys, h].double().t().contiguous()
        vh = v[keys, h].double().contiguous()
        qh = q[rows, h].double() / math.sqrt(dim)
        for i in range(0, len(rows), step):
            out[i:i + step, h] = torch.softmax(qh[i:i + step] @ kt, dim=1) @ vh
    return out


def _blend(a, b, weight):
    return (1.0 - weight) * a.double() + weight * b.double()


def exact(case, seed):
    t, kind, T = _draws(case, seed), case["kind"], case["T"]
    if kind == "select":
        x = t["latents"].double().transpose(1, 2).reshape(case["B"], T, -1).contiguous()
        x = x / x.norm(dim=2, keepdim=True).clamp_min(1e-8)
        return torch.stack([e @ e.t().contiguous() for e in x])
    key = _frames(T, case["M"])
    other = [f for f in range(T) if f not in key]
    projected = None
    if kind in ("step", "project"):
        z = t["latents"]
        projected = z[:, 1].double().clone()
        for f in other:
            projected[:, :, f] = _blend(z[:, 0, :, f], z[:, 1, :, f], (TIMES[0] - TIMES[2]) / (TIMES[0] - TIMES[1]))
        if kind == "project":
            return projected
    N = case["H"] * case["W"]
    tokens = torch.arange(T * N, device="cuda").view(T, N)
    if kind == "cache":
        frame = [t[n].view(T, N * case["heads"] * case["dim"]) for n in ("h0", "h1", "k", "v")]
        store = torch.stack([frame[0][other], frame[1][other]], dim=1).double().reshape(-1)
        weight = (T_WARM - T_SKIP) / (T_WARM - T_RHYTHMIC + 1e-8)
        k, v = frame[2].double(), frame[3].double()
        k[other] = v[other] = _blend(frame[0][other], frame[1][other], weight)
        return store, k.view(t["k"].shape), v.view(t["v"].shape)
    rows = tokens[key].reshape(-1)
    out = _attention(t["q"], t["k"], t["v"], rows, rows if kind == "mask" else tokens.reshape(-1))
    if kind != "step":
        return out
    full = t["full"].double()
    full[rows] = out
    return projected, out, full
