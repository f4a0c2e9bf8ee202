"""The key-block-major forward and backward at the edges of their cuts: every number of partials per chunk of
the merges, rows that end inside a chunk, blocks in parts, queries with fewer kept blocks than top-k, lists
shorter and longer than a step, slices worked through together and one after the other."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# (batch, heads, kv_heads, N, d, B, k).  Partials per query, (k + 1) x parts: 1 2 3 4 | 5 6 | 8 9 | 10 11 | 13 | 17 33 65
@pytest.mark.parametrize("batch,heads,kv,N,d,B,k", [
    (1, 2, 0, 1024, 64, 32, 0), (1, 1, 0, 1024, 64, 64, 1), (1, 2, 0, 960, 64, 96, 2), (1, 2, 0, 2048, 64, 128, 3),
    (1, 2, 0, 1024, 128, 32, 4), (1, 2, 0, 2048, 64, 256, 2), (1, 3, 0, 2048, 128, 64, 7), (1, 8, 0, 2048, 64, 128, 8),
    (2, 8, 4, 2048, 128, 128, 4), (1, 2, 0, 2048, 64, 64, 10), (1, 2, 0, 2048, 64, 32, 12), (1, 16, 0, 2048, 64, 64, 16),
    (1, 2, 0, 4096, 128, 64, 32), (1, 1, 0, 4096, 64, 32, 64), (1, 1, 0, 32, 64, 32, 3), (1, 1, 0, 128, 64, 128, 8)])
def test_key_major_against_the_plain_kernels(batch, heads, kv, N, d, B, k):
    import paper_2511_11571_amd as moba
    b = moba.binding
    g = torch.Generator(device="cuda").manual_seed(31 * k + N + d)
    hkv = kv or heads
    Q, K, V, dO = (torch.randn((batch, h, N, d), generator=g, device="cuda").to(torch.bfloat16)
                   for h in (heads, hkv, hkv, heads))
    shape = lambda flags: moba.Shape(batch, heads, N, d, B, k, 0, b.BF16, 0.0, flags, kv)  # noqa: E731
    km, plain = shape(b.FLAG_KEY_MAJOR), shape(b.FLAG_REFERENCE_KERNELS)
    _, cent = moba.centroids(km, K)
    idx, lists = moba.topk(km, Q, cent)
    # partials that no query fills hold whatever the workspace held
    ws = [torch.full((x,), 0xff, dtype=torch.uint8, device="cuda") for x in moba.workspace_bytes(km)[1:]]
    O, lse = moba.forward(km, Q, K, V, idx, lists, ws=ws[0])
    got = moba.backward(km, Q, K, V, O, lse, dO, idx, lists, ws=ws[1])
    plists = moba.build_lists(plain, idx)
    rO, rlse = moba.forward(plain, Q, K, V, idx, plists)
    ref = moba.backward(plain, Q, K, V, rO, rlse, dO, idx, plists)
    # fp32 sums of the same bf16 products in another order
    assert float((lse - rlse).abs().max()) < 1e-4
    # P, the partials and the result are rounded to bf16 (2^-9 each at most); gradients: P, dS, the partials
    # and the result, and D from rounded O
    for x, y in zip((O,) + tuple(got), (rO,) + tuple(ref)):
        x, y = x.float(), y.float()
        assert bool(torch.isfinite(x).all())
        assert float((x - y).norm() / y.norm()) < 2 ** -7


def test_forward_partials_are_divided_with_one_rounding():
    """Scores of zero: the probabilities are 1 and a query's only partial is sum / count, with whole numbers above and
    below.  The reciprocal of the count is a correctly rounded one, which shows where the quotient lies half-way
    between two bf16 values or next to it."""
    import numpy as np
    import paper_2511_11571_amd as moba
    b = moba.binding
    for d, B in ((64, 128), (64, 96), (128, 64)):
        heads = 2048
        sh = moba.Shape(1, heads, B, d, B, 0, 0, b.BF16, 0.0, b.FLAG_KEY_MAJOR, 0)
        g = torch.Generator(device="cuda").manual_seed(B)
        Q = torch.zeros((1, heads, B, d), dtype=torch.bfloat16, device="cuda")
        V = torch.randint(0, 256, Q.shape, generator=g, device="cuda").to(torch.bfloat16)
        idx = torch.empty((1, heads, B, 0), dtype=torch.int32, device="cuda")
        O, _ = moba.forward(sh, Q, Q, V, idx, moba.build_lists(sh, idx))
        inv = np.float32(1) / np.arange(1, B + 1, dtype=np.float32)
        total = V.cpu().double().cumsum(2).numpy().astype(np.float32)             # exact
        want = torch.from_numpy(total * inv[:, None]).to(torch.bfloat16)
        assert torch.equal(O.cpu(), want)
