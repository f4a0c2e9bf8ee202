"""The key convolution's backward on workspaces of every size it takes: chunks of 16, 32, 64 and 128 rows, sequences
that end inside a chunk's first rows, inside its last ones and with it."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,heads,N,d,W,dtype", [
    (1, 2, 4096, 128, 4, "bf16"), (2, 1, 2048 + 32, 128, 3, "f32"), (1, 3, 8192 + 96, 64, 8, "bf16"), (1, 1, 32, 64, 4, "bf16"),
    (2, 2, 4096, 64, 1, "f32")])
def test_every_workspace_gives_the_same_gradients(batch, heads, N, d, W, dtype):
    import paper_2511_11571_amd as moba
    b = moba.binding
    code, dt = (b.BF16, torch.bfloat16) if dtype == "bf16" else (b.F32, torch.float32)
    sh = moba.Shape(batch, heads, N, d, 32, 2, W, code)
    g = torch.Generator(device="cuda").manual_seed(N + W)
    K, G = (torch.randn((batch, heads, N, d), generator=g, device="cuda").to(dt) for _ in range(2))
    w = 0.5 * torch.randn((heads, d, W), generator=g, device="cuda")
    full = ctypes.c_size_t(0)
    assert b.lib().moba_key_conv_backward_workspace(ctypes.byref(sh.c()), ctypes.byref(full)) == 0
    slices, per = batch * heads, 4 * W * d
    wgs = lambda rows: -(-(-(-N // rows)) // (2048 // d))  # noqa: E731
    sizes = [(slices * wgs(rows) * per + 255) // 256 * 256 + 256 for rows in (16, 32, 64, 128)]
    assert full.value in sizes
    out = []
    for size in sorted(set(sizes)):
        if size <= full.value:
            ws = torch.full((size,), 0xff, dtype=torch.uint8, device="cuda")
            out.append(moba.key_conv_backward(sh, K, w, G, ws=ws))
    dK, dw = out[0]                                       # chunks of 128 rows
    for x, y in out[1:]:
        # a row of dK is the same sum wherever its chunk starts; dw: fp32 sums of N terms in another order
        assert torch.equal(x, dK)
        assert float((y - dw).norm() / dw.norm()) < 1e-5
    with pytest.raises(Exception):
        moba.key_conv_backward(sh, K, w, G, ws=torch.empty(min(sizes) - 256, dtype=torch.uint8, device="cuda"))
    # against the definition in 64 bits
    Kd, wd, Gd = K.double().requires_grad_(), w.double().requires_grad_(), G.double()
    a = sum(wd[None, :, None, :, lag] * torch.nn.functional.pad(Kd, (0, 0, lag, 0))[:, :, :N] for lag in range(W))
    ((Kd + torch.nn.functional.silu(a)) * Gd).sum().backward()
    tol = 2 ** -8 if dtype == "bf16" else 1e-5             # dK is stored in the I/O type
    assert float((dK.double() - Kd.grad).norm() / Kd.grad.norm()) < tol
    assert float((dw.double() - wd.grad).norm() / wd.grad.norm()) < 1e-5
