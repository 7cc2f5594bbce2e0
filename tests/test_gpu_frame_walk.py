"""The walk over a frame list's keys where key tiles run from one listed frame
into the next: frames just under, at and above a tile, neighbours and gaps, each
form of the kernel (whole tiles, split tail, small launches). Frames that are not
listed hold NaN, so a key taken from one spoils the result. Against fp64 on the
GPU, a head at a time, with the bf16 gates."""
import math

import numpy as np
import pytest
import torch

from paper_2606_06309_amd import workloads
from parity import assert_parity, torch_bf16_to_f64

pytestmark = pytest.mark.gpu

rf = pytest.importorskip("paper_2606_06309_amd.binding")


def _reference(q, k, v, rows, keys):
    out = np.empty((len(rows), q.shape[1], q.shape[2]))
    for h in range(q.shape[1]):
        kt = k[keys, h].double().t().contiguous()
        s = q[rows, h].double() / math.sqrt(q.shape[2]) @ kt
        out[:, h] = (torch.softmax(s, dim=1) @ v[keys, h].double().contiguous()).cpu().numpy()
    return out


def _run(T, H, W, heads, d, qf, kvf, forms):
    w = workloads.custom(T, H, W, heads, d, qf, dtype="bf16", seed=T * W + d)
    q, k, v = workloads.make_qkv(w, device="cuda")
    tok = torch.arange(w.S, device="cuda").view(T, w.N)
    rows, keys = tok[list(qf)].reshape(-1), tok[list(kvf)].reshape(-1)
    ref = _reference(q, k, v, rows, keys)
    masked = [f for f in range(T) if f not in kvf]
    k.view(T, -1)[masked] = float("nan")
    v.view(T, -1)[masked] = float("nan")
    need = rf.rf_attention_workspace(len(qf), len(kvf), T, H, W, heads, d, rf.RF_BF16)
    shared = rf.attention_shares_keys(len(qf), len(kvf), T, H, W, heads, d, rf.RF_BF16)
    for form in forms:
        assert form == "whole" or shared == (form == "small")
        print(f"[case] frame walk T={T} N={w.N} heads={heads} d={d} kv={kvf} {form}", flush=True)
        if form == "whole":
            out = rf.rf_frame_attention(q, k, v, qf, kvf, T, H, W)
        else:
            ws = torch.full((max(need, 64),), 0x7f, dtype=torch.uint8, device="cuda")
            out = rf.rf_frame_attention(q, k, v, qf, kvf, T, H, W, workspace=ws)
            assert bool((ws == 0x7f).all()) == (form == "small")
        assert_parity(torch_bf16_to_f64(out), ref, "bf16", form)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kvf", [(0, 2, 5), (1, 2, 3), (0, 1, 4, 6), (6,)], ids=lambda f: "-".join(map(str, f)))
@pytest.mark.parametrize("hw", [(1, 31), (1, 32), (5, 7), (7, 9), (8, 8), (5, 13), (1, 127), (8, 16), (3, 43), (10, 23)],
                         ids=lambda n: f"N{n[0] * n[1]}")
def test_small_sizes(hw, kvf, d):
    _run(7, *hw, 2, d, (0, 4), kvf, ("whole", "small"))


@pytest.mark.parametrize("case", [(13, 20, 30, 12, 128, (0, 4, 8, 12), (0, 1, 2, 4, 7, 8, 11, 12)),
                                  (15, 16, 31, 12, 64, (0, 3, 6, 9, 12), (0, 2, 3, 5, 6, 8, 9, 11, 12, 14))],
                         ids=["d128", "d64"])
def test_split_tail(case):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("sized for 256 compute units")
    _run(*case, ("whole", "split"))


def test_split_tail_that_stays_frame_aligned():
    """32 frames of 65 keys are 33 tiles end to end but 64 frame-aligned ones, for which the plan has 8 parts:
    33 tiles in parts of five would leave the eighth without one, so the parts stay frame-aligned."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("sized for 256 compute units")
    kvf = tuple(f for f in range(33) if f != 7)
    plan = rf.rf_attention_plan(33, 32, 33, 5, 13, 32, 128, rf.RF_BF16)
    assert (plan["tail_tiles"], plan["parts"], plan["key_tiles_per_part"]) == (32, 8, 8)
    _run(33, 5, 13, 32, 128, tuple(range(33)), kvf, ("whole", "split"))
