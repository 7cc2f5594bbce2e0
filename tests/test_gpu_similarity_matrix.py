"""rf_frame_similarity on the matrix cores at the edges of its tiling: frame
counts around the 4-frame blocks up to the 64 of the matrix-core path and past
it, planes around the 64-element chunks and at every alignment, fewer chunks
than waves, and batches past the workgroup target, in both types.

The bound: a Gram entry is a sum of n products of two rounded-exactly values,
each product rounded at most once and added in some order, so its error is at
most n 2^-53 sum |x_i x_j| <= n 2^-53 |x_i| |x_j|; each norm contributes half
that relative error and the root, product and quotient a few 2^-53 more."""
import pytest
import torch

pytestmark = pytest.mark.gpu

rf = pytest.importorskip("paper_2606_06309_amd.binding")

CASES = [(1, 3, T, 9, 7) for T in (1, 2, 3, 4, 5, 8, 9, 13, 16, 17, 21, 25, 29, 33, 36, 40, 41, 45, 49, 53, 57, 61,
                                   63, 64, 65)]
CASES += [(1, 2, 6, 1, W) for W in (1, 2, 3, 5, 62, 63, 64, 65, 66, 67, 127, 129, 191, 4099)]
CASES += [(5, 1, 11, 5, 13), (3, 16, 33, 34, 62), (513, 1, 3, 2, 3), (2, 7, 64, 33, 65)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_against_fp64(shape, dtype):
    B, C, T, H, W = shape
    print(f"[case] similarity {shape} {dtype}", flush=True)
    g = torch.Generator().manual_seed(B * 1000 + T * 10 + W)
    x = (torch.randn(shape, generator=g) + 0.5 * torch.randn((B, C, 1, H, W), generator=g)).to(dtype)
    got = rf.rf_frame_similarity(x.cuda()).cpu()
    f = x.double().transpose(1, 2).reshape(B, T, -1).contiguous()
    norm = f.norm(dim=2).clamp_min(1e-8)
    ref = torch.bmm(f, f.transpose(1, 2).contiguous()) / (norm[:, :, None] * norm[:, None, :])
    assert got.shape == ref.shape
    bound = 2 * (2 * C * H * W + 16) * 2.0 ** -53      # this sum's and the reference's
    assert (got - ref).abs().max().item() <= bound
    assert torch.equal(got, got.transpose(1, 2))
    assert (got.diagonal(dim1=1, dim2=2) - 1).abs().max().item() <= 4 * 2.0 ** -53


def test_a_frame_without_numbers_spoils_only_its_own_entries():
    x = torch.randn((1, 2, 7, 5, 13), generator=torch.Generator().manual_seed(5))
    clean = rf.rf_frame_similarity(x.cuda()).cpu()
    x[0, 1, 2, 4, 12] = float("nan")
    x[0, :, 5] = 0.0
    got = rf.rf_frame_similarity(x.cuda()).cpu()
    keep = [0, 1, 3, 4, 6]
    assert torch.equal(got[0][keep][:, keep], clean[0][keep][:, keep])
    assert torch.isnan(got[0, 2]).all() and torch.isnan(got[0, :, 2]).all()
    assert bool((got[0, 5][keep + [5]] == 0).all())


@pytest.mark.parametrize("T", [33, 36, 37])
@pytest.mark.parametrize("h", [127, 129])
def test_batches_on_both_sides_of_the_long_walk(T, h):
    """4 videos of 16 x h x 128: 16,256 and 16,512 chunks of 64 elements, around 16 a wave at one workgroup
    per compute unit; 36 frames are the most that then take two."""
    g = torch.Generator().manual_seed(T * h)
    x = torch.randn((4, 16, T, h, 128), generator=g)
    print(f"[case] similarity long walk T={T} h={h}", flush=True)
    out = rf.rf_frame_similarity(x.cuda()).cpu()
    e = x.double().transpose(1, 2).reshape(4, T, -1)
    e = e / e.norm(dim=2, keepdim=True)
    for b in range(4):
        assert float((out[b] - e[b] @ e[b].t().contiguous()).abs().max()) < 16 * h * 128 * 2.0 ** -52
