"""fp32 attention on the matrix cores: sizes around the edges of its tiles (32 and 64 keys, 128 and 32 query
rows), both ways a launch is cut (with a workspace small launches share out the keys of a tile), frame lists,
and scores of -inf. Against the fp64 oracle within the fp32 gates."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_06309_amd import workloads
from parity import assert_parity

pytestmark = pytest.mark.gpu

rf = pytest.importorskip("paper_2606_06309_amd.binding")


def _f64(t):
    return t.cpu().numpy().astype(np.float64)


def _ws():
    return torch.empty(16, dtype=torch.uint8, device="cuda")   # fp32 takes none: any buffer will do


def _shares(w, mkv=None):
    """Whether the launch given a workspace shares out the keys (one without a workspace never does)."""
    return rf.attention_shares_keys(w.M, mkv or w.T, w.T, w.H, w.W, w.heads, w.head_dim, rf.RF_F32)


# (T, H, W, heads, keyframes): keys 1, 31..33, 63..65, 127..129; query rows from 1 to 390; one wave's
# key tile (32), one per wave (128 or 256) and one more than that
CASES = [(1, 1, 1, 3, (0,)), (1, 1, 31, 2, (0,)), (1, 4, 8, 2, (0,)), (1, 3, 11, 2, (0,)), (3, 3, 7, 2, (0, 2)),
         (2, 4, 8, 1, (1,)), (5, 1, 13, 2, (0, 4)), (1, 127, 1, 1, (0,)), (2, 8, 8, 2, (0, 1)), (3, 1, 43, 2, (0, 1, 2)),
         (5, 10, 13, 3, (0, 2, 4)), (9, 5, 13, 65, (3,))]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"S{c[0] * c[1] * c[2]}x{c[3]}")
def test_tile_edges(case, d):
    T, H, W, heads, kf = case
    w = workloads.custom(T, H, W, heads, d, kf, dtype="f32", seed=70)
    print(f"[case] {w}", flush=True)
    q, k, v = workloads.make_qkv(w, device="cuda")
    ref = oracle.keyframe_attention(q.cpu(), k.cpu(), v.cpu(), kf, w.N)
    assert _shares(w)
    whole = rf.rf_keyframe_attention(q, k, v, kf, T, H, W)
    split = rf.rf_keyframe_attention_ws(q, k, v, kf, T, H, W, workspace=_ws())
    assert_parity(_f64(whole), ref, "f32", "whole tiles")
    assert_parity(_f64(split), ref, "f32", "shared keys")
    # the allocation-free call is cut as the workspace call; whole tiles give a row the same
    # bits in a launch of every frame
    assert torch.equal(rf.rf_keyframe_attention_noalloc(q, k, v, kf, T, H, W), split)
    everything = rf.rf_keyframe_attention(q, k, v, range(T), T, H, W)
    assert torch.equal(everything.view(T, w.N, heads, d)[list(kf)].reshape(whole.shape), whole)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N", [(1, 31), (1, 33), (5, 13), (10, 13)], ids=lambda n: f"N{n[0] * n[1]}")
def test_frame_lists(N, d):
    H, W = N
    w = workloads.custom(6, H, W, 2, d, (0, 3, 5), dtype="f32", seed=71)
    q, k, v = workloads.make_qkv(w, device="cuda")
    kv = (1, 2, 5)
    assert _shares(w, len(kv))
    ref = oracle.frame_attention(q.cpu(), k.cpu(), v.cpu(), w.keyframes, kv, w.N)
    k[0:w.N] = float("nan")   # a frame that is not listed is never read
    for ws in (None, _ws()):
        out = rf.rf_frame_attention(q, k, v, w.keyframes, kv, w.T, H, W, workspace=ws)
        assert_parity(_f64(out), ref, "f32", f"list, workspace {ws is not None}")


@pytest.mark.parametrize("d", [64, 128])
def test_keys_with_scores_of_minus_infinity_count_nothing(d):
    """Keys whose scores are -inf for every query (here the first 40, so a whole key tile and part of the
    next) leave the softmax over the others."""
    w = workloads.custom(4, 4, 20, 2, d, (0, 2), dtype="f32", seed=72)
    q, k, v = workloads.make_qkv(w, device="cuda")
    q[..., 0] = 1.0
    k[..., 0] = 0.0
    k[:40, :, 0] = -float("inf")
    assert _shares(w)
    qd, kd, vd = (x.double().transpose(0, 1).contiguous() for x in (q, k[40:], v[40:]))
    rows = torch.cat([torch.arange(f * w.N, (f + 1) * w.N) for f in w.keyframes]).cuda()
    ref = torch.softmax(qd[:, rows] @ kd.transpose(1, 2).contiguous() / d ** 0.5, dim=2) @ vd
    ref = ref.transpose(0, 1).cpu().numpy()
    for out in (rf.rf_keyframe_attention(q, k, v, w.keyframes, w.T, w.H, w.W),
                rf.rf_keyframe_attention_ws(q, k, v, w.keyframes, w.T, w.H, w.W, workspace=_ws())):
        assert_parity(_f64(out), ref, "f32", "-inf scores")
