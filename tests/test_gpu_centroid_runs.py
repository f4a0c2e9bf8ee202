"""Centroids and key conv where a lane group's rows are taken in batches of 16, 8, 4 and 1: run lengths with every
remainder, blocks of one run and of several, idle lane groups in the last workgroup, copies with and without a filter."""
import pytest
import torch

import paper_2511_11571_amd as moba
from paper_2511_11571_amd import binding

pytestmark = pytest.mark.gpu

# (batch, heads, blocks, d, B): rows per run 7, 25, 12, 16, 31, 29, 16, 43
SHAPES = [(1, 1, 3, 64, 7), (1, 2, 5, 64, 100), (3, 3, 5, 64, 96), (1, 1, 1, 64, 128), (2, 1, 4, 64, 31), (1, 5, 2, 128, 58),
          (1, 3, 3, 128, 64), (1, 1, 9, 128, 172)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("W", [0, 1, 3, 4, 8])
@pytest.mark.parametrize("batch,heads,n,d,B", SHAPES)
def test_centroids_of_runs_with_remainders(batch, heads, n, d, B, W, dtype):
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator().manual_seed(B * 10 + W)
    N = n * B
    K = torch.randn(batch, heads, N, d, generator=g).to(t)
    w = torch.randn(heads, d, W, generator=g) if W else None
    shape = moba.Shape(batch, heads, N, d, B, 1, W, binding.BF16 if dtype == "bf16" else binding.F32)
    Keff = torch.full_like(K, 9.0).cuda()
    Keff, cent = moba.centroids(shape, K.cuda(), w.cuda() if W else None, Keff)
    assert cent.shape == (batch, heads, n, d)
    got, cent = Keff.cpu(), cent.double().cpu()
    if W == 0:
        assert torch.equal(got, K)
        alone = moba.centroids(shape, K.cuda())[1].double().cpu()
        assert torch.equal(alone, cent)
    else:
        x, a = K.double(), torch.zeros(batch, heads, N, d, dtype=torch.float64)
        mag = torch.zeros_like(a)
        for l in range(W):
            rows = torch.nn.functional.pad(x, (0, 0, l, 0))[:, :, :N]
            a += w[None, :, None, :, l].double() * rows
            mag += (w[None, :, None, :, l].double() * rows).abs()
        want = x + a * torch.sigmoid(a)
        # W roundings of a (|d silu / da| < 1.1); the sigmoid's exp rounds its argument, a quarter of |a| at most counts,
        # and with the reciprocal adds a few units; then the sum's and the type's rounding
        bound = (1.1 * W * 2.0 ** -24 * mag + (4 + a.abs() / 4) * 2.0 ** -23 * a.abs() + 2.0 ** -24 * want.abs()
                 + (2.0 ** -8 if dtype == "bf16" else 2.0 ** -24) * want.abs())
        assert ((got.double() - want).abs() <= bound + 1e-30).all()
    blocks = got.double().view(batch, heads, n, B, d)
    # B - 1 additions of fp32 and a division
    assert ((cent - blocks.mean(3)).abs() <= (B + 1) * 2.0 ** -24 * blocks.abs().mean(3)).all()


# (slices, n, d, B, W): calls that take another number of rows together than their slices on their own (2^19 lanes and
# more; with a filter 2^16), and their neighbours: runs of 16, 32, 8 and 8 rows of d = 64, 14 in one, 16 and 32 of d = 128
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("slices,n,d,B,W", [(8, 1024, 64, 128, 0), (8, 1024, 64, 256, 0), (8, 1024, 64, 64, 0), (8, 2048, 64, 32, 0),
                                            (8, 8192, 64, 14, 0), (16, 512, 128, 64, 0), (16, 512, 128, 128, 3), (8, 128, 128, 128, 2),
                                            (8, 128, 128, 124, 4), (8, 1024, 64, 32, 1)])
def test_centroids_of_a_call_and_of_its_slices(slices, n, d, B, W, dtype):
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    code = binding.BF16 if dtype == "bf16" else binding.F32
    g = torch.Generator(device="cuda").manual_seed(n + B)
    K = torch.randn((1, slices, n * B, d), generator=g, device="cuda").to(t)
    w = torch.randn((slices, d, W), generator=g, device="cuda") if W else None
    whole = moba.centroids(moba.Shape(1, slices, n * B, d, B, 1, W, code), K, w, torch.full_like(K, 9.0))
    part = moba.Shape(1, 1, n * B, d, B, 1, W, code)
    # a run's rows are filtered and added one after the other, however many of them are requested together: the same bits
    for s in range(slices):
        ws = w[s:s + 1].contiguous() if W else None
        Keff, cent = moba.centroids(part, K[:, s:s + 1].contiguous(), ws, torch.full_like(K[:, :1], 9.0))
        assert torch.equal(whole[0][:, s:s + 1], Keff) and torch.equal(whole[1][:, s:s + 1], cent)
    if W == 0:
        assert torch.equal(whole[0], K)
