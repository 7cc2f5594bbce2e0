"""Keys whose scores are -inf for every query, or as low as masked scores are set
to where -inf is avoided, leave the softmax over the other keys, wherever a walk
over the keys begins with whole tiles of them: the first tiles of a whole-tile
launch, of every part of a split tail, of each wave of a small launch, of a frame
list and of the cache form. Against fp64 over the keys that count, with the bf16
gates; the query rows and keys hold no other special values. And scores that are
all the same large number, whose product with the scale is exact: every key counts
the same."""
import math

import numpy as np
import pytest
import torch

from paper_2606_06309_amd import workloads
from parity import assert_parity, torch_bf16_to_f64

pytestmark = pytest.mark.gpu

rf = pytest.importorskip("paper_2606_06309_amd.binding")

TILE = {64: 128, 128: 64}   # keys per tile of 256 query rows
LOWEST = torch.finfo(torch.bfloat16).min
VALUES = pytest.mark.parametrize("value", [-float("inf"), LOWEST, -1e20], ids=["inf", "lowest", "1e20"])


def _inputs(w, dropped, value):
    """q, k, v of w with every score against the keys `dropped` at `value` (v is as drawn there)."""
    q, k, v = workloads.make_qkv(w, device="cuda")
    q[..., 0] = 1.0
    k[..., 0] = 0.0
    k[dropped, :, 0] = value
    return q, k, v


def _check(out, w, q, k, v, keys, what):
    rows = torch.cat([torch.arange(f * w.N, (f + 1) * w.N) for f in w.keyframes])
    ref = np.empty((len(rows), w.heads, w.head_dim))
    for h in range(w.heads):
        s = q[rows, h].double() / math.sqrt(w.head_dim) @ k[keys, h].double().t().contiguous()
        ref[:, h] = (torch.softmax(s, dim=1) @ v[keys, h].double().contiguous()).cpu().numpy()
    assert_parity(torch_bf16_to_f64(out), ref, "bf16", what)


def _counted(order, dropped):
    gone = set(dropped.tolist())
    return torch.tensor([t for t in order.tolist() if t not in gone])


@VALUES
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("tiles", [1, 2, 3])
def test_whole_tiles(tiles, d, value):
    """The first `tiles` key tiles and a few keys more (the loop takes its tiles two at a time)."""
    w = workloads.custom(5, 10, 13, 2, d, (0, 2), dtype="bf16", seed=91)
    dropped = torch.arange(tiles * TILE[d] + 9)
    print(f"[case] {value} whole tiles d={d} tiles={tiles}", flush=True)
    q, k, v = _inputs(w, dropped, value)
    out = rf.rf_keyframe_attention(q, k, v, w.keyframes, w.T, w.H, w.W)
    _check(out, w, q, k, v, _counted(torch.arange(w.S), dropped), "whole tiles")


@VALUES
@pytest.mark.parametrize("case", [(21, 16, 16, 12, 64, (0, 5, 10, 15, 20)), (13, 16, 16, 12, 128, (0, 4, 8, 12))],
                         ids=["d64", "d128"])
def test_parts_of_a_split_tail(case, value):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("sized for 256 compute units")
    T, H, W, heads, d, kf = case
    w = workloads.custom(T, H, W, heads, d, kf, dtype="bf16", seed=92)
    plan = rf.rf_attention_plan(w.M, T, T, H, W, heads, d, rf.RF_BF16)
    assert plan["parts"] > 1
    step = plan["key_tiles_per_part"] * TILE[d]
    starts = [p * step for p in range(plan["parts"])]
    dropped = torch.cat([torch.arange(s, min(s + TILE[d] + 9, w.S)) for s in starts])
    print(f"[case] {value} split tail {case}", flush=True)
    q, k, v = _inputs(w, dropped, value)
    ws = torch.full((plan["workspace_bytes"],), 0x7f, dtype=torch.uint8, device="cuda")
    out = rf.rf_keyframe_attention_ws(q, k, v, kf, T, H, W, workspace=ws)
    assert not bool((ws == 0x7f).all())
    _check(out, w, q, k, v, _counted(torch.arange(w.S), dropped), "split tail")


@VALUES
@pytest.mark.parametrize("workspace", [False, True], ids=["whole", "split"])
@pytest.mark.parametrize("case", [(13, 20, 30, 12, 128, (0, 4, 8, 12), (0, 1, 2, 4, 7, 8, 11, 12)),
                                  (15, 16, 31, 12, 64, (0, 3, 6, 9, 12), (0, 2, 3, 5, 6, 8, 9, 11, 12, 14))],
                         ids=["d128", "d64"])
def test_frame_lists(case, workspace, value):
    """The first tiles of the list's keys, and those around the middle where the second of two parts begins
    (the walk end to end and the frame-aligned one put it a tile or two apart)."""
    if workspace and torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("sized for 256 compute units")
    T, H, W, heads, d, kf, kvf = case
    w = workloads.custom(T, H, W, heads, d, kf, dtype="bf16", seed=93)
    order = torch.arange(w.S).view(T, w.N)[list(kvf)].reshape(-1)
    tile, n = TILE[d], len(order)
    half = -(-n // tile) // 2
    dropped = torch.cat([order[:tile + 9], order[(half - 2) * tile:(half + 5) * tile]])
    print(f"[case] {value} frame list {case} workspace={workspace}", flush=True)
    q, k, v = _inputs(w, dropped, value)
    ws = None
    if workspace:
        plan = rf.rf_attention_plan(w.M, len(kvf), T, H, W, heads, d, rf.RF_BF16)
        assert plan["parts"] == 2
        ws = torch.empty(plan["workspace_bytes"], dtype=torch.uint8, device="cuda")
    out = rf.rf_frame_attention(q, k, v, kf, kvf, T, H, W, workspace=ws)
    _check(out, w, q, k, v, _counted(order, dropped), "frame list")


@VALUES
@pytest.mark.parametrize("d", [64, 128])
def test_cache_form(d, value):
    """Frame 0, a keyframe, begins with scores of -inf; the other frames' keys are projected states."""
    w = workloads.custom(5, 16, 16, 2, d, (0, 2), dtype="bf16", seed=94)
    dropped = torch.arange(TILE[d] + 9)
    print(f"[case] {value} cache form d={d}", flush=True)
    q, k, v = _inputs(w, dropped, value)
    nk = [f for f in range(w.T) if f not in w.keyframes]
    D = w.heads * w.head_dim
    store = torch.zeros(rf.rf_cache_store_bytes(len(nk), w.N, D, w.torch_dtype) // 2, dtype=w.torch_dtype, device="cuda")
    h0, h1 = (workloads.make_hidden(w, i, device="cuda") for i in (0, 1))
    cache = rf.rf_cache_init(nk, w.T, w.N, D, w.torch_dtype, 40.0, store=store, h_full=h0)
    rf.rf_cache_shift_store(cache, 37.0, store=store, h_full=h1)
    out = rf.rf_keyframe_attention_cached(q, k, v, w.keyframes, w.T, w.H, w.W, cache, store, 38.0)
    rf.rf_cache_project_kv(cache, store, k, v, 38.0)
    _check(out, w, q, k, v, _counted(torch.arange(w.S), dropped), "cache form")


@VALUES
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("frames", [None, (0, 1, 3, 4)], ids=["dense", "list"])
def test_waves_of_a_small_launch(frames, d, value):
    """Whole first tiles of some of the eight waves, whole second tiles of others."""
    w = workloads.custom(5, 10, 13, 2, d, (0, 2), dtype="bf16", seed=95)
    dropped = torch.arange(64, 64 + 320)
    print(f"[case] {value} small launch d={d} frames={frames}", flush=True)
    q, k, v = _inputs(w, dropped, value)
    ws = torch.empty(16, dtype=torch.uint8, device="cuda")
    assert rf.attention_shares_keys(w.M, len(frames or range(w.T)), w.T, w.H, w.W, w.heads, d, rf.RF_BF16)
    if frames:
        out = rf.rf_frame_attention(q, k, v, w.keyframes, frames, w.T, w.H, w.W, workspace=ws)
    else:
        out = rf.rf_keyframe_attention_ws(q, k, v, w.keyframes, w.T, w.H, w.W, workspace=ws)
    order = torch.arange(w.S).view(w.T, w.N)[list(frames or range(w.T))].reshape(-1)
    _check(out, w, q, k, v, _counted(order, dropped), "small launch")


@pytest.mark.parametrize("value", [-1e6, -2.0 ** 40, 2.0 ** 40, -2.0 ** 100], ids=["-1e6", "-2^40", "2^40", "-2^100"])
@pytest.mark.parametrize("d", [64, 128])
def test_equal_scores_of_any_size(d, value):
    """The mean of v, from whole tiles, a small launch and a split tail."""
    several = (20, 30 if d == 64 else 20, (0, 4, 8, 12, 16), "split")
    for T, heads, kf, form in ((5, 2, (0, 2), "whole"), (5, 2, (0, 2), "small"), several):
        w = workloads.custom(T, 10, 13, heads, d, kf, dtype="bf16", seed=96)
        print(f"[case] equal scores {value} d={d} {form}", flush=True)
        q, k, v = workloads.make_qkv(w, device="cuda")
        q[..., 0] = 1.0
        k.zero_()
        k[..., 0] = value
        if form == "whole":
            out = rf.rf_keyframe_attention(q, k, v, kf, T, w.H, w.W)
        else:
            if torch.cuda.get_device_properties(0).multi_processor_count == 256:
                assert rf.attention_shares_keys(w.M, T, T, w.H, w.W, heads, d, rf.RF_BF16) == (form == "small")
                assert form == "small" or rf.rf_attention_plan(w.M, T, T, w.H, w.W, heads, d, rf.RF_BF16)["parts"] > 1
            out = rf.rf_keyframe_attention_ws(q, k, v, kf, T, w.H, w.W)
        ref = v.double().mean(dim=0).cpu().numpy()[None].repeat(w.M * w.N, axis=0)
        assert_parity(torch_bf16_to_f64(out), ref, "bf16", form)
