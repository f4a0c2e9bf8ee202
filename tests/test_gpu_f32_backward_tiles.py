"""The fp32 backward whose waves own a 16-key tile each, at the sizes where it can go wrong: a last tile of few keys, a part of
few keys behind whole ones, shares without rows, one share, no kept blocks, shared heads, both types; each gradient by itself;
and infinities and NaN among the keys at d = 128."""
import pytest
import torch

import paper_2511_11571_amd as moba
from paper_2511_11571_amd import binding

pytestmark = pytest.mark.gpu

#        dtype   d   B   blocks  k  heads kv
CASES = [("f32", 64, 49, 20, 4, 2, 0), ("f32", 128, 64, 24, 3, 2, 1), ("bf16", 128, 50, 12, 4, 2, 0), ("f32", 64, 114, 9, 3, 4, 2),
         ("f32", 128, 114, 9, 0, 1, 0), ("f32", 64, 64, 1, 0, 1, 0), ("bf16", 64, 62, 300, 2, 12, 0), ("f32", 64, 64, 16, 2, 200, 0),
         # many shares of few short walks, several slices to an XCD
         ("f32", 64, 64, 8, 7, 1, 0), ("f32", 128, 64, 9, 8, 2, 0), ("f32", 64, 64, 24, 5, 24, 0)]


@pytest.mark.parametrize("odd", [False, True])
@pytest.mark.parametrize("dtype,d,B,n,k,heads,kv", CASES)
def test_against_the_plain_kernels(dtype, d, B, n, k, heads, kv, odd):
    N, code, hkv = B * n, binding.F32 if dtype == "f32" else binding.BF16, kv or heads
    dt = torch.float32 if code == binding.F32 else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(d + B + n)
    Q, K, V, dO = (torch.randn((1, h, N, d), generator=g, device="cuda").to(dt) for h in (heads, hkv, hkv, heads))
    sh, plain = (moba.Shape(1, heads, N, d, B, k, 0, code, 0.0, f, kv) for f in (0, binding.FLAG_REFERENCE_KERNELS))
    _, cent = moba.centroids(sh, K)
    idx, lists = moba.topk(sh, Q, cent)
    if odd:                                              # in the last block, which no other query keeps
        V[:, :, N - B // 2, 3], K[:, :, N - B // 2 + 1, 5] = float("inf"), float("nan")
    O, lse = moba.forward(plain, Q, K, V, idx, moba.build_lists(plain, idx))
    want = moba.backward(plain, Q, K, V, O, lse, dO, idx, moba.build_lists(plain, idx))
    ws = torch.full((moba.workspace_bytes(sh)[2],), 0xff, dtype=torch.uint8, device="cuda")        # (NaN)
    got = moba.backward(sh, Q, K, V, O, lse, dO, idx, lists, ws=ws)
    # fp32 sums of up to B (k + 1) products in another order; bf16 results: two roundings of 2^-9 and a fp32 sum
    tol = 1e-5 if dtype == "f32" else 2 ** -7
    for name, a, b in list(zip(("dQ", "dK", "dV"), got, want))[:1 if odd else 3]:
        a, b = a.double(), b.double()
        seen = torch.isfinite(b)
        assert torch.equal(torch.isfinite(a), seen), name
        assert bool(seen.all()) != odd, name
        assert float((a - b)[seen].norm() / b[seen].norm()) < tol, name
    if odd:
        return
    out = tuple(torch.full_like(x, 7.0) for x in got)
    call = lambda parts: moba.backward(sh, Q, K, V, O, lse, dO, idx, lists, ws=ws, out=out, parts=parts)  # noqa: E731
    call(binding.BWD_PREPROCESS)
    call(binding.BWD_DQ)
    assert torch.equal(out[0], got[0]) and all(bool((x == 7.0).all()) for x in out[1:])
    out[0].fill_(7.0)
    call(binding.BWD_DKDV)
    assert bool((out[0] == 7.0).all()) and torch.equal(out[1], got[1]) and torch.equal(out[2], got[2])
