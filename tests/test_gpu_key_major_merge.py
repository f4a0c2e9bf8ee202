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


# Limits of the relative errors (2-norms) against 64 bits.  Roundings to bf16 of P, of a partial and of the result (O); of dS, of
# a partial and of the result (dQ); of dS (dK) or P (dV) and the result; D from rounded O.  With normally distributed inputs they
# come to 2.6e-3, 2.9e-3, 2.5e-3 and 2.4e-3; with one bit less in any single one of them, at least one of the four
# comes to 3.6e-3, 3.9e-3, 3.7e-3 and 3.5e-3 or more (the same roundings carried out in 64 bits on the CPU).
LIMITS = {"O": 3.0e-3, "dQ": 3.3e-3, "dK": 2.9e-3, "dV": 2.8e-3}


@pytest.mark.parametrize("heads,kv,N,d,B,k", [
    (2, 0, 2048, 64, 128, 8), (1, 0, 2016, 64, 96, 10), (2, 1, 2048, 128, 64, 16), (1, 0, 2048, 64, 256, 4),
    (1, 0, 2048, 128, 256, 3), (1, 0, 2048, 64, 32, 12)])
def test_key_major_errors_against_64_bits(heads, kv, N, d, B, k):
    import paper_2511_11571_amd as moba
    b = moba.binding
    g = torch.Generator(device="cuda").manual_seed(N + d + k)
    hkv = kv or heads
    Q, K, V, dO = (torch.randn((1, h, N, d), generator=g, device="cuda").to(torch.bfloat16) for h in (heads, hkv, hkv, heads))
    sh = moba.Shape(1, heads, N, d, B, k, 0, b.BF16, 0.0, b.FLAG_KEY_MAJOR, kv)
    _, cent = moba.centroids(sh, K)
    idx, lists = moba.topk(sh, Q, cent)
    O, lse = moba.forward(sh, Q, K, V, idx, lists)
    dQ, dK, dV = moba.backward(sh, Q, K, V, O, lse, dO, idx, lists)
    t = torch.arange(N, device="cuda") // B
    causal = torch.ones((N, N), dtype=torch.bool, device="cuda").tril()
    want = {"O": [], "lse": [], "dQ": [], "dK": [], "dV": []}
    for h in range(heads):
        q, kk, v, do = Q[0, h].double(), K[0, h * hkv // heads].double(), V[0, h * hkv // heads].double(), dO[0, h].double()
        kept = (idx[0, h, :, :, None] == torch.arange(N // B, device="cuda")).any(1)
        seen = kept.repeat_interleave(B, 1) | (causal & (t[:, None] == t[None]))
        s = (q @ kk.T / d ** 0.5).masked_fill(~seen, -float("inf"))
        L = torch.logsumexp(s, 1)
        p = (s - L[:, None]).exp()
        o = p @ v
        ds = p * (do @ v.T - (do * o).sum(1)[:, None]) / d ** 0.5
        for name, x in (("O", o), ("lse", L), ("dQ", ds @ kk), ("dK", ds.T @ q), ("dV", p.T @ do)):
            want[name].append(x)
    want = {name: torch.stack(x) for name, x in want.items()}
    if kv:
        want["dK"], want["dV"] = (want[x].view(hkv, heads // hkv, N, d).sum(1) for x in ("dK", "dV"))
    for name, x in (("O", O), ("dQ", dQ), ("dK", dK), ("dV", dV)):
        assert float((x[0].double() - want[name]).norm() / want[name].norm()) < LIMITS[name], name
    # scores of about 4 units of log2 or less in fp32, sums of at most 2^11 terms in a few stages, one logarithm
    assert float((lse[0].double() - want["lse"]).pow(2).mean().sqrt()) < 2.0 ** -20


# (heads, N, d, B, k): slices that an XCD takes together, forward / backward, of those it has: 4 / 2 of 4, 3 / 3 of 3, 2 / 1 of
# 4, 3 / 1 of 3
@pytest.mark.parametrize("heads,N,d,B,k", [(32, 4096, 128, 128, 2), (24, 4096, 64, 128, 3), (32, 8192, 128, 128, 2), (24, 5376, 128, 64, 2)])
def test_slices_worked_through_together_give_what_each_gives_alone(heads, N, d, B, k):
    import paper_2511_11571_amd as moba
    b = moba.binding
    g = torch.Generator(device="cuda").manual_seed(heads + N)
    Q, K, V, dO = (torch.randn((1, heads, N, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(4))

    def step(Q, K, V, dO):
        sh = moba.Shape(1, Q.shape[1], N, d, B, k, 0, b.BF16, 0.0, b.FLAG_KEY_MAJOR, 0)
        _, cent = moba.centroids(sh, K)
        idx, lists = moba.topk(sh, Q, cent)
        # (partials that nothing fills are NaN)
        ws = [torch.full((x,), 0xff, dtype=torch.uint8, device="cuda") for x in moba.workspace_bytes(sh)[1:]]
        O, lse = moba.forward(sh, Q, K, V, idx, lists, ws=ws[0])
        return (O, lse) + tuple(moba.backward(sh, Q, K, V, O, lse, dO, idx, lists, ws=ws[1]))

    whole = step(Q, K, V, dO)
    for h in range(0, heads, 8):                           # one slice per XCD
        part = step(*(x[:, h:h + 8].contiguous() for x in (Q, K, V, dO)))
        for x, y in zip(whole, part):
            assert bool(torch.isfinite(y.float()).all()) and torch.equal(x[:, h:h + 8], y)
