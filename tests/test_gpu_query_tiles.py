"""The query-tile forward and backward at the edges of a tile's row lists: lists of 1 to 256 rows that end
anywhere inside a group of sixteen or four, blocks that no row keeps, more pairs than one set of lists holds,
last tiles with few rows; what a key with a NaN leaves to the rows that do not attend it."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def skewed_routing(batch, heads, N, B, k, seed):
    """Up to k past blocks per row: block j with a weight that falls off with j, a quarter of the rows with less
    than k, every seventh block with none."""
    g = torch.Generator().manual_seed(seed)
    n = N // B
    past = torch.arange(N)[:, None] // B > torch.arange(n)[None, :]
    past &= (torch.arange(n) % 7 != 3)[None, :]
    w = torch.rand((batch, heads, N, n), generator=g).log() * (1.0 + torch.arange(n) / 4.0)
    w = torch.where(past, w, torch.tensor(-float("inf")))
    val, idx = w.topk(min(k, n), dim=-1)
    drop = torch.rand((batch, heads, N, 1), generator=g) < 0.25
    few = torch.randint(0, k + 1, (batch, heads, N, 1), generator=g)
    keep = torch.isfinite(val) & (~drop | (torch.arange(min(k, n)) < few))
    idx = torch.where(keep, idx, torch.tensor(n)).sort(dim=-1).values
    out = torch.full((batch, heads, N, k), -1, dtype=torch.int32)
    out[..., :min(k, n)] = torch.where(idx < n, idx, torch.tensor(-1)).to(torch.int32)
    return out


# (batch, heads, kv_heads, N, d, B, k)
@pytest.mark.parametrize("batch,heads,kv,N,d,B,k", [
    (1, 2, 0, 1024, 64, 32, 5), (1, 2, 0, 1056, 64, 32, 8), (1, 1, 0, 4096, 64, 32, 72), (2, 2, 1, 1088, 64, 64, 4),
    # lists of 30, 45 and 248 rows on average (the kernels for short ones end at 48, forward, and 128, dQ; above: 72, 88, 206, B = 64: 87)
    (1, 2, 0, 1024, 64, 32, 2), (1, 2, 0, 1024, 64, 32, 3), (1, 1, 0, 1024, 64, 32, 31),
    (1, 2, 0, 960, 64, 96, 3), (1, 2, 0, 1024, 128, 32, 7), (1, 4, 2, 1312, 128, 32, 12), (1, 1, 0, 8320, 128, 64, 130)])
def test_query_tiles_against_the_plain_kernels(batch, heads, kv, N, d, B, k):
    import paper_2511_11571_amd as moba
    b = moba.binding
    g = torch.Generator(device="cuda").manual_seed(17 * k + N + d)
    hkv = kv or heads
    Q, K, V, dO = (torch.randn((batch, h, N, d), generator=g, device="cuda").to(torch.bfloat16)
                   for h in (heads, hkv, hkv, heads))
    shape = lambda flags: moba.Shape(batch, heads, N, d, B, k, 0, b.BF16, 0.0, flags, kv)  # noqa: E731
    tiles, plain = shape(b.FLAG_QUERY_TILES), shape(b.FLAG_REFERENCE_KERNELS)
    hidx = skewed_routing(batch, heads, N, B, k, 3 * N + k)
    idx = hidx.cuda()
    lists, plists = moba.build_lists(tiles, idx), moba.build_lists(plain, idx)
    O, lse = moba.forward(tiles, Q, K, V, idx, lists)
    got = moba.backward(tiles, Q, K, V, O, lse, dO, idx, lists)
    rO, rlse = moba.forward(plain, Q, K, V, idx, plists)
    ref = moba.backward(plain, Q, K, V, rO, rlse, dO, idx, plists)
    # fp32 sums of the same bf16 products in another order
    assert float((lse - rlse).abs().max()) < 1e-4
    # P and the result are rounded to bf16 (2^-9 each at most); gradients: P, dS and the result, and D from rounded O
    for x, y in zip((O,) + tuple(got), (rO,) + tuple(ref)):
        x, y = x.float(), y.float()
        assert bool(torch.isfinite(x).all())
        assert float((x - y).norm() / y.norm()) < 2 ** -7
    # the sums are integers: a key's NaN reaches the rows that attend it and changes no bit of another row
    u = N // 3
    bad = K.clone()
    bad[0, 0, u, 1] = float("nan")
    t = torch.arange(N)
    attends = ((hidx[0, 0] == u // B).any(-1) | ((t // B == u // B) & (t >= u))).cuda()
    nO, nlse = moba.forward(tiles, Q, bad, V, idx, lists)
    assert bool(torch.isnan(nO[0, 0][attends]).all()) and bool(torch.isnan(nlse[0, 0][attends]).all())
    assert torch.equal(nO[0, 0][~attends], O[0, 0][~attends]) and torch.equal(nlse[0, 0][~attends], lse[0, 0][~attends])
