"""fp32 attention on the matrix cores at the block sizes where its tiles of 16 keys and its key splits can go
wrong: blocks below a tile, one over a tile, beyond what one workgroup holds, no kept blocks, the longest
rows, shared heads."""
import numpy as np
import pytest
import torch

import paper_2511_11571_amd as moba
from paper_2511_11571_amd import binding
from tests import parity

pytestmark = pytest.mark.gpu

#        d   B    blocks  k  heads kv
CASES = [(64, 8, 40, 3, 2, 0), (64, 17, 12, 4, 1, 0), (128, 24, 9, 0, 1, 0), (64, 50, 8, 3, 4, 2),
         (128, 96, 5, 2, 2, 1), (64, 128, 4, 2, 1, 0), (128, 200, 4, 3, 1, 0), (64, 8, 80, 64, 1, 0)]


@pytest.mark.parametrize("d,B,n,k,heads,kv", CASES)
def test_fp32_forward_and_backward(oracle, d, B, n, k, heads, kv):
    N, hkv = B * n, kv or heads
    g = torch.Generator().manual_seed(9000 + B)
    Q, dO = (torch.randn((1, heads, N, d), generator=g) for _ in range(2))
    K, V = (torch.randn((1, hkv, N, d), generator=g) for _ in range(2))
    sh = moba.Shape(1, heads, N, d, B, k, 0, binding.F32, 0.0, 0, kv)
    Q64, K64, V64, dO64 = (x.double().numpy()[0] for x in (Q, K, V, dO))
    Ke, Ve = (oracle.gqa_expand(x, heads, hkv) for x in (K64, V64))
    kept, _ = oracle.topk(Q64, oracle.centroids(Ke, B), B, k)
    idx = torch.from_numpy(kept).reshape(1, heads, N, k).cuda()
    lists = moba.build_lists(sh, idx)
    Qd, Kd, Vd, dOd = (x.cuda() for x in (Q, K, V, dO))
    O, lse = moba.forward(sh, Qd, Kd, Vd, idx, lists)
    got = (O, *moba.backward(sh, Qd, Kd, Vd, O, lse, dOd, idx, lists))
    rO, rlse = oracle.attn_fwd(Q64, Ke, Ve, kept, B, 1.0 / np.sqrt(d))
    rQ, rK, rV = oracle.attn_bwd(Q64, Ke, Ve, kept, dO64, B, 1.0 / np.sqrt(d))
    want = (rO, rQ, oracle.gqa_reduce(rK, heads, hkv), oracle.gqa_reduce(rV, heads, hkv))
    assert parity.max_abs(lse.double().cpu().numpy()[0], rlse) < parity.LSE_TOL["f32"]
    for name, a, b in zip(("O", "dQ", "dK", "dV"), got, want):
        assert parity.rel_l2(a.double().cpu().numpy()[0], b) < parity.GRAD_TOL["f32"], name


@pytest.mark.parametrize("dtype,d,B,n,k,kv", [("f32", 64, 32, 24, 5, 0), ("f32", 128, 96, 6, 3, 1), ("bf16", 64, 50, 12, 4, 0)])
def test_lists_without_places(dtype, d, B, n, k, kv):
    """Lists built for kernels that file nothing by the place of a block (here: the plain ones) hold no places:
    attention finds them in the rows of kept blocks, and the results are the same bit for bit."""
    N, heads, code = B * n, 2, binding.F32 if dtype == "f32" else binding.BF16
    g = torch.Generator(device="cuda").manual_seed(d + B)
    Q, K, V, dO = (torch.randn((1, h, N, d), generator=g, device="cuda").to(torch.float32 if code == binding.F32 else torch.bfloat16)
                   for h in (heads, kv or heads, kv or heads, heads))
    sh = moba.Shape(1, heads, N, d, B, k, 0, code, 0.0, 0, kv)
    plain = moba.Shape(1, heads, N, d, B, k, 0, code, 0.0, binding.FLAG_REFERENCE_KERNELS, kv)
    _, cent = moba.centroids(sh, K)
    idx, lists = moba.topk(sh, Q, cent)
    bare = moba.build_lists(plain, idx)
    R = int(lists[0][0, 0, -1])
    assert bool((lists[1][..., :R] >> 24 > 0).any()) and bool((bare[1][..., :R] >> 24 == 0).all())
    out = []
    for some in (lists, bare):
        ws = [torch.full((size,), 0xff, dtype=torch.uint8, device="cuda") for size in moba.workspace_bytes(sh)]  # (NaN)
        O, lse = moba.forward(sh, Q, K, V, idx, some, ws=ws[1])
        out.append((O, lse, *moba.backward(sh, Q, K, V, O, lse, dO, idx, some, ws=ws[2])))
    for a, b in zip(*out):
        assert torch.equal(a, b)


@pytest.mark.parametrize("dtype,d,B,n,k,kv", [("f32", 64, 64, 12, 3, 0), ("f32", 128, 96, 6, 2, 1), ("bf16", 64, 50, 8, 3, 0)])
def test_keys_that_a_query_does_not_see_cannot_reach_it(dtype, d, B, n, k, kv):
    """Infinities and NaN in keys and values: a query's output and gradient are finite exactly where the plain
    kernels, which touch nothing but the keys that a query sees, find them finite, and equal there."""
    N, heads, code = B * n, 2, binding.F32 if dtype == "f32" else binding.BF16
    dt, hkv = torch.float32 if code == binding.F32 else torch.bfloat16, kv or heads
    g = torch.Generator(device="cuda").manual_seed(3 * d + B)
    Q, K, V, dO = (torch.randn((1, h, N, d), generator=g, device="cuda").to(dt) for h in (heads, hkv, hkv, heads))
    Q[..., 0] = Q[..., 0].abs() + 0.5
    shapes = [moba.Shape(1, heads, N, d, B, k, 0, code, 0.0, f, kv) for f in (0, binding.FLAG_REFERENCE_KERNELS)]
    _, cent = moba.centroids(shapes[0], K)
    idx, _ = moba.topk(shapes[0], Q, cent)
    inf, last = float("inf"), (n - 1) * B
    # in the last block, which no other query keeps; and keys of no weight, among them a block's first
    V[:, :, last + B // 2, 3], K[:, :, last + B // 2 + 1, 5], V[:, :, last + B - 1, 9] = inf, float("nan"), float("nan")
    K[:, :, 2 * B:3 * B:7, 0] = -inf
    out = []
    for sh in shapes:
        lists = moba.build_lists(sh, idx)
        O, lse = moba.forward(sh, Q, K, V, idx, lists)
        out.append((O, lse, moba.backward(sh, Q, K, V, O, lse, dO, idx, lists)[0]))
    tol = 1e-5 if dtype == "f32" else 2 ** -7              # fp32 sums in another order; two roundings to bf16
    for name, a, b in zip(("O", "lse", "dQ"), *out):
        a, b = a.double(), b.double()
        seen = torch.isfinite(b)
        assert torch.equal(torch.isfinite(a), seen), name
        assert not bool(seen.all()) and float(seen.double().mean()) > 0.4, name
        assert float((a - b)[seen].norm() / b[seen].norm()) < tol, name
