"""The decode call where its selection and its cut over workgroups change: short rows of kept blocks at the edges of
the groups that bound them, ties, scores that are no numbers; queries shared by several workgroups, workspaces of any
content, replays of a captured graph."""
import ctypes

import pytest
import torch

import paper_2511_11571_amd as moba
from paper_2511_11571_amd import binding
from tests import parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("levels", [3, 40, 10 ** 6])
@pytest.mark.parametrize("past,k", [(2, 1), (17, 16), (63, 5), (64, 16), (65, 16), (200, 17), (1024, 8), (1025, 1), (4095, 16), (4096, 15)])
def test_kept_blocks_of_exact_scores(past, k, levels):
    """Scores that fp32 sums give exactly (whole numbers, one channel): the kept blocks are the first k by score, ties
    to the lower block -- with many ties (more of them than are ranked directly), some, and hardly any."""
    heads, B, d = 3, 2, 64
    g = torch.Generator().manual_seed(past * 31 + k + levels)
    Q = torch.zeros((1, heads, 1, d))
    Q[..., 7] = torch.tensor([1.0, -1.0, 2.0])[None, :, None]
    cent = torch.zeros((1, heads, past, d))
    cent[..., 7] = torch.randint(-levels, levels + 1, (1, heads, past), generator=g).float()
    N = past * B + 1
    K = torch.randn((1, heads, N, d), generator=g)
    sh = moba.Shape(1, heads, N, d, B, k, 0, binding.BF16)
    to = lambda x: x.to(torch.bfloat16).cuda()  # noqa: E731
    _, _, idx = moba.decode_forward(sh, 1, to(Q), to(K), to(K), cent.cuda())
    score = (Q[..., 7] * cent[..., 7])[0]
    best = score.sort(dim=-1, descending=True, stable=True).indices[:, :k].sort(-1).values
    assert torch.equal(idx[0, :, 0].cpu().long(), best)


def test_scores_that_are_no_numbers():
    """Infinite scores and NaN: k blocks, ascending; the infinite ones first, as with longer rows."""
    past, B, d, k = 300, 2, 64, 6
    Q = torch.ones((1, 1, 1, d))
    cent = torch.randn((1, 1, past, d), generator=torch.Generator().manual_seed(1))
    cent[0, 0, [11, 250]] = float("inf")
    cent[0, 0, 40] = -float("inf")
    sh = moba.Shape(1, 1, past * B + 1, d, B, k, 0, binding.BF16)
    K = torch.zeros((1, 1, past * B + 1, d), dtype=torch.bfloat16).cuda()
    for nan in (False, True):
        if nan:
            cent[0, 0, 99, 0] = float("nan")
        idx = moba.decode_forward(sh, 1, Q.to(torch.bfloat16).cuda(), K, K, cent.cuda())[2][0, 0, 0].cpu()
        z = cent.sum(-1)[0, 0]
        finite = z.masked_fill(~torch.isfinite(z), -float("inf")).sort(descending=True).indices
        assert bool((idx.diff() > 0).all()) and {11, 250} <= set(idx.tolist()) and 40 not in idx.tolist()
        assert set(idx.tolist()) - {11, 99, 250} <= set(finite[:k - 2].tolist())


def _case(batch, heads, kv, N, d, B, k, q_len, dtype):
    dt = torch.bfloat16 if dtype == binding.BF16 else torch.float32
    g = torch.Generator(device="cuda").manual_seed(N + k)
    hkv = kv or heads
    Q, K, V = (torch.randn(s, generator=g, device="cuda").to(dt) for s in
               ((batch, heads, q_len, d), (batch, hkv, N, d), (batch, hkv, N, d)))
    past = (N - 1) // B
    cent = K[:, :, :past * B].reshape(batch, hkv, past, B, d).mean(3, dtype=torch.float32).contiguous()
    return moba.Shape(batch, heads, N, d, B, k, 0, dtype, 0.0, 0, kv), Q, K, V, cent


# (batch, heads, kv_heads, N, d, B, k, q_len, dtype), workgroups per query: keys that do not divide among them, blocks that no
# load instruction fills, one block that a query's shares all lie in, last shares that are shorter
SHARED = [((1, 1, 0, 9011, 64, 128, 32, 1, binding.BF16), 8), ((1, 4, 2, 5003, 64, 64, 65, 1, binding.BF16), 8), ((1, 4, 0, 3001, 128, 100, 13, 3, binding.BF16), 2),
          ((1, 2, 1, 4100, 128, 33, 40, 4, binding.BF16), 4), ((2, 8, 0, 2500, 64, 64, 32, 2, binding.F32), 4), ((2, 16, 4, 5000, 64, 256, 14, 2, binding.BF16), 2),
          ((1, 1, 0, 4097, 64, 4096, 1, 1, binding.BF16), 8), ((1, 3, 0, 3203, 128, 16384, 0, 1, binding.BF16), 8), ((1, 4, 1, 2100, 128, 50, 20, 1, binding.F32), 8)]


def _call(sh, q_len, Q, K, V, cent, O, lse, ws):
    f = binding.lib().moba_decode_forward_ws
    ptr = lambda t: ctypes.c_void_p(0 if t is None else t.data_ptr())  # noqa: E731
    assert f(ctypes.byref(sh.c()), q_len, ptr(Q), ptr(K), ptr(V), ptr(cent), cent.shape[2], ptr(O), ptr(lse), None, ptr(ws),
             ctypes.c_size_t(0 if ws is None else ws.numel()), ctypes.c_void_p(binding._stream())) == 0


@pytest.mark.parametrize("case,workgroups", SHARED)
def test_shared_queries(case, workgroups):
    """Against one workgroup per query, and bit for bit from call to call whatever the workspace held."""
    q_len, dtype = case[7], case[8]
    sh, Q, K, V, cent = _case(*case)
    need = binding._decode_workspace_bytes(sh, q_len)
    assert _workgroups(sh, q_len) == workgroups
    one = torch.empty_like(Q), torch.empty(Q.shape[:3], device="cuda")
    _call(sh, q_len, Q, K, V, cent, *one, None)
    first = None
    for fill in (0xff, 0, 0x5a, None):                        # None: what the call before left
        ws = torch.full((need,), fill, dtype=torch.uint8, device="cuda") if fill is not None else ws
        O, lse = torch.empty_like(Q), torch.empty(Q.shape[:3], device="cuda")
        _call(sh, q_len, Q, K, V, cent, O, lse, ws)
        if first is None:
            first = O, lse
        assert torch.equal(O, first[0]) and torch.equal(lse, first[1])
    # the same fp32 terms added up in another order (at most 4200, in chains of under 300 terms: 300 x 2^-24 = 2e-5), O rounded once
    assert float((lse - one[1]).abs().max()) < 1e-4
    name = "bf16" if dtype == binding.BF16 else "f32"
    assert float((O.float() - one[0].float()).abs().max()) < parity.O_TOL[name] / 2
    O, lse, _ = moba.decode_forward(sh, q_len, Q, K, V, cent)
    assert torch.equal(O, first[0]) and torch.equal(lse, first[1])


def _infinite_values(heads, N, d, B, k, keys):
    """Queries that attend all N keys, keys[c] with an infinite value in channel c: infinite exactly there, as every
    key's weight is positive, and the other channels as without."""
    assert (N - 1) // B <= k and len(keys) < d
    sh, Q, K, V, cent = _case(1, heads, 0, N, d, B, k, 1, binding.BF16)
    want, lse, _ = moba.decode_forward(sh, 1, Q, K, V, cent)
    for c, key in enumerate(keys):
        V[0, :, key, c] = float("inf")
    got = moba.decode_forward(sh, 1, Q, K, V, cent)
    assert torch.equal(got[1], lse)
    assert bool((got[0][..., :len(keys)] == float("inf")).all()), got[0][..., :len(keys)]
    assert torch.equal(got[0][..., len(keys):], want[..., len(keys):])


@pytest.mark.parametrize("heads,N,d,B,k,workgroups", [(1, 4001, 64, 128, 31, 4), (1, 1999, 128, 64, 31, 4), (40, 4001, 64, 128, 31, 2),
                                                      (1, 4100, 64, 128, 32, 8)])
def test_infinite_values_of_every_share(heads, N, d, B, k, workgroups):
    """... in two keys from the middle of each workgroup's share (whole load instructions of 512 / d keys)."""
    each = -(-N // (workgroups * 512 // d)) * (512 // d)
    assert workgroups == _workgroups(_shape(1, heads, 0, N, d, B, k, 1, binding.BF16), 1)
    _infinite_values(heads, N, d, B, k, [each * w + each // 2 + i for w in range(workgroups) for i in (0, 5)])


@pytest.mark.parametrize("heads,N,d,B,k,workgroups", [(1, 4001, 64, 128, 31, 4), (1, 4100, 64, 128, 32, 8), (40, 2013, 128, 33, 60, 2), (1, 1999, 128, 64, 31, 4),
                                                      (3, 700, 64, 64, 10, 1), (2, 1000, 128, 33, 30, 1)])
def test_infinite_values_around_the_ends_of_shares(heads, N, d, B, k, workgroups):
    """... in the last and first keys of shares, of the own block and of the sequence: rows that a neighbour's last loads read too."""
    each = -(-N // (workgroups * 512 // d)) * (512 // d)
    assert workgroups == _workgroups(_shape(1, heads, 0, N, d, B, k, 1, binding.BF16), 1)
    edges = [each * w + i for w in range(1, workgroups) for i in (-1, 0, 5)] + [(N - 1) // B * B, N - 2, N - 1]
    _infinite_values(heads, N, d, B, k, sorted(set(edges)))


def test_shared_queries_in_a_graph():
    sh, Q, K, V, cent = _case(*SHARED[1][0])
    eager = moba.decode_forward(sh, 1, Q, K, V, cent, want_idx=False)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        moba.decode_forward(sh, 1, Q, K, V, cent, want_idx=False)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        O, lse, _ = moba.decode_forward(sh, 1, Q, K, V, cent, want_idx=False)
    for _ in range(5):
        O.zero_()
        lse.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(O, eager[0]) and torch.equal(lse, eager[1])
        moba.decode_forward(sh, 1, Q, K, V, cent, want_idx=False)


def test_workspace_sizes():
    need = lambda *a: binding._decode_workspace_bytes(_shape(*a), a[7])  # noqa: E731
    assert need(2, 16, 0, 131109, 64, 128, 8, 1, binding.BF16) == 0           # little to read
    assert need(8, 16, 0, 30000, 128, 64, 32, 1, binding.BF16) == 0           # many queries
    sh = _shape(*SHARED[0][0])
    n = binding._decode_workspace_bytes(sh, 1)
    one = ctypes.c_void_p(256)                                                # (never dereferenced: refused on the host)
    assert binding.lib().moba_decode_forward_ws(ctypes.byref(sh.c()), 1, one, one, one, one, 70, one, one, None, one,
                                                ctypes.c_size_t(n - 1), None) == -3


def _workgroups(sh, q_len):
    """Workgroups per query, from the size of the workspace: a counter per query, rounded up, and d + 2 floats a workgroup."""
    need, queries = binding._decode_workspace_bytes(sh, q_len), sh.batch * sh.heads * q_len
    return max(1, (need - (8 * queries + 255) // 256 * 256) // (queries * (sh.head_dim + 2) * 4))


def _shape(batch, heads, kv, N, d, B, k, q_len, dtype):
    return moba.Shape(batch, heads, N, d, B, k, 0, dtype, 0.0, 0, kv)
