"""The gradients one call at a time on key-block-major shapes: dQ alone, dK and dV alone, both together."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# (heads, kv_heads, N, d, B, k): a 32-key group to four of them per workgroup, parts of larger blocks, shared heads
@pytest.mark.parametrize("heads,kv_heads,N,d,B,k", [
    (2, 0, 4096, 64, 32, 2), (2, 0, 4096, 64, 64, 3), (3, 0, 4032, 64, 96, 4), (2, 0, 4096, 64, 128, 4),
    (2, 0, 4096, 64, 256, 2), (2, 0, 4096, 128, 64, 4), (4, 2, 4096, 128, 128, 3)])
def test_parts_agree_with_the_whole_backward(heads, kv_heads, N, d, B, k):
    import paper_2511_11571_amd as moba
    b = moba.binding
    g = torch.Generator(device="cuda").manual_seed(5)
    hkv = kv_heads or heads
    Q, K, V, dO = (torch.randn((1, h, N, d), generator=g, device="cuda").to(torch.bfloat16)
                   for h in (heads, hkv, hkv, heads))
    sh = moba.Shape(1, heads, N, d, B, k, 0, b.BF16, 0.0, 0, kv_heads)
    Ke, cent = moba.centroids(sh, K)
    idx, lists = moba.topk(sh, Q, cent)
    O, lse = moba.forward(sh, Q, Ke, V, idx, lists)
    whole = moba.backward(sh, Q, Ke, V, O, lse, dO, idx, lists)
    ws = torch.empty(moba.workspace_bytes(sh)[2], dtype=torch.uint8, device="cuda")
    out = tuple(torch.full_like(x, 7.0) for x in whole)
    call = lambda parts: moba.backward(sh, Q, Ke, V, O, lse, dO, idx, lists, ws=ws, out=out, parts=parts)  # noqa: E731
    call(b.BWD_PREPROCESS)
    call(b.BWD_DQ)
    assert all(bool((x == 7.0).all()) for x in out[1:])
    assert torch.equal(out[0], whole[0])                 # the same sums in the same order
    out[0].fill_(7.0)
    call(b.BWD_DKDV)
    assert bool((out[0] == 7.0).all())
    for x, y in zip(out[1:], whole[1:]):
        # fp32 sums of the same bf16 P and dS in another order, each stored in bf16: two roundings of 2^-9
        assert float((x.float() - y.float()).norm() / y.float().norm()) < 2 ** -8
