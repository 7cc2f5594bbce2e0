"""The bf16 attention of small launches (32 query rows a workgroup, the keys
shared out among its eight waves): sizes at the edges of the row tile and of the
key tile, fewer key tiles than waves, one and several a wave, ragged frames in
the frame-list form, and maxima that move late in every wave's keys. Against the
fp64 oracle with the bf16 gates. Which launches take it the plan says; the
workspace, which a split tail fills, is left alone."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_06309_amd import workloads
from parity import assert_parity, torch_bf16_to_f64

pytestmark = pytest.mark.gpu

rf = pytest.importorskip("paper_2606_06309_amd.binding")

# T, H, W, heads, keyframes: rows M*H*W around 32, keys T*H*W around the 32- and
# 64-key tiles and around eight of them
CASES = [
    (3, 1, 31, 1, (1,)), (3, 1, 32, 2, (0,)), (3, 1, 33, 3, (0, 2)),
    (2, 3, 43, 1, (0,)), (4, 8, 8, 2, (0, 3)), (4, 1, 127, 1, (0, 2)), (2, 16, 16, 5, (1,)),
    (3, 1, 171, 1, (0,)), (9, 10, 13, 3, (0, 4, 8)), (9, 17, 31, 5, (0, 4, 8)),
]


def _shares(w, mkv=None):
    return rf.attention_shares_keys(w.M, mkv or w.T, w.T, w.H, w.W, w.heads, w.head_dim, rf.RF_BF16)


def _run(w, kvf=None, scale_k=None, small=True):
    assert _shares(w, len(kvf) if kvf else None) == small
    q, k, v = workloads.make_qkv(w, device="cuda")
    if scale_k is not None:
        k = (k.float() * scale_k).to(k.dtype)
    n = rf.rf_attention_workspace(w.M, len(kvf) if kvf else w.T, w.T, w.H, w.W, w.heads, w.head_dim, rf.RF_BF16)
    ws = torch.full((max(n, 64),), 0x7f, dtype=torch.uint8, device="cuda")
    if kvf:
        out = rf.rf_frame_attention(q, k, v, w.keyframes, kvf, w.T, w.H, w.W, workspace=ws)
        ref = oracle.frame_attention(q.cpu(), k.cpu(), v.cpu(), w.keyframes, kvf, w.N)
    else:
        out = rf.rf_keyframe_attention_ws(q, k, v, w.keyframes, w.T, w.H, w.W, workspace=ws)
        ref = oracle.keyframe_attention(q.cpu(), k.cpu(), v.cpu(), w.keyframes, w.N)
    assert_parity(torch_bf16_to_f64(out), ref, "bf16", w.name)
    return bool((ws == 0x7f).all())


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"T{c[0]}_N{c[1] * c[2]}_h{c[3]}")
def test_edges(case, d):
    T, H, W, heads, kf = case
    print(f"[case] small attention {case} d={d}", flush=True)
    assert _run(workloads.custom(T, H, W, heads, d, kf, dtype="bf16", seed=T * W + d))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N", [(1, 33), (10, 13), (16, 16)], ids=lambda n: f"N{n[0] * n[1]}")
def test_frame_list(N, d):
    w = workloads.custom(11, *N, 3, d, (0, 4, 10), dtype="bf16", seed=81 + d)
    print(f"[case] small frame list N={N} d={d}", flush=True)
    assert _run(w, kvf=(0, 1, 3, 4, 6, 10))


@pytest.mark.parametrize("d", [64, 128])
def test_late_maxima(d):
    w = workloads.custom(9, 10, 13, 3, d, (0, 4, 8), dtype="bf16", seed=82)
    ramp = torch.from_numpy(np.linspace(0.25, 5.0, w.S, dtype=np.float32)).cuda()[:, None, None]
    print(f"[case] small late maxima d={d}", flush=True)
    assert _run(w, scale_k=ramp)


@pytest.mark.parametrize("T", [5, 17])
@pytest.mark.parametrize("d", [64, 128])
def test_waves_that_begin_with_scores_of_minus_infinity(d, T):
    """Keys 128..319 score -inf for every query: whole first tiles of some of the eight waves, whole second
    tiles of others, none of the first 128 keys. They leave the softmax over the other keys. At 17 frames the
    plan splits, so a workspace left alone shows that the plan did not run."""
    w = workloads.custom(T, 10, 13, 2, d, (0, 2), dtype="bf16", seed=84)
    assert _shares(w)
    parts = rf.rf_attention_plan(w.M, w.T, w.T, w.H, w.W, w.heads, d, rf.RF_BF16)["parts"]
    assert T == 5 or parts > 1
    q, k, v = workloads.make_qkv(w, device="cuda")
    q[..., 0] = 1.0
    k[..., 0] = 0.0
    k[128:320, :, 0] = -float("inf")
    print(f"[case] small -inf scores d={d}", flush=True)
    ws = torch.full((max(rf.rf_attention_workspace(w.M, w.T, w.T, w.H, w.W, w.heads, d, rf.RF_BF16), 64),), 0x7f,
                    dtype=torch.uint8, device="cuda")
    out = rf.rf_keyframe_attention_ws(q, k, v, w.keyframes, w.T, w.H, w.W, workspace=ws)
    assert bool((ws == 0x7f).all())
    counted = torch.cat([torch.arange(128), torch.arange(320, w.S)])
    rows = torch.cat([torch.arange(f * w.N, (f + 1) * w.N) for f in w.keyframes])
    qd, kd, vd = (x.cpu()[i].double().transpose(0, 1).contiguous() for x, i in ((q, rows), (k, counted), (v, counted)))
    ref = torch.softmax(qd @ kd.transpose(1, 2).contiguous() / d ** 0.5, dim=2) @ vd
    assert_parity(torch_bf16_to_f64(out), ref.transpose(0, 1).numpy(), "bf16", "-inf scores")


@pytest.mark.parametrize("case", [(21, 16, 16, 12, 64, (0, 5, 10, 15, 20)), (13, 16, 16, 12, 128, (0, 4, 8, 12))],
                         ids=["d64", "d128"])
def test_above_the_rule_the_tail_is_split(case):
    T, H, W, heads, d, kf = case
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("sized for 256 compute units")
    print(f"[case] split above the small rule {case}", flush=True)
    assert not _run(workloads.custom(T, H, W, heads, d, kf, dtype="bf16", seed=83), small=False)
