"""The gate's kernels at the borders of their dispatch: blocks that fill a tile of 16 or spill one over,
the last block counts whose scores stay in registers and the first that do not, the lengths of row on both
sides of each rule, fp32 up to and beyond its limit, equal scores.  The two sweeps run on calls of 300000 query rows
and more only: those have tests of their own, against the exact search, with shared key/value heads, packed
batches, and strips that are searched again because too many scores are equal."""
import numpy as np
import pytest
import torch

import paper_2511_11571_amd as moba
from paper_2511_11571_amd import binding
from tests import parity

pytestmark = pytest.mark.gpu

#        dtype   d   blocks  k   B
CASES = [("bf16", 64, 1, 1, 2), ("bf16", 64, 16, 1, 3), ("bf16", 64, 17, 16, 2), ("bf16", 128, 18, 64, 2),
         ("bf16", 64, 320, 64, 2), ("bf16", 64, 321, 64, 2), ("bf16", 64, 321, 16, 2), ("bf16", 64, 512, 16, 2),
         ("bf16", 64, 513, 16, 3), ("bf16", 64, 1000, 1, 2), ("bf16", 64, 2047, 12, 2), ("bf16", 128, 256, 64, 2),
         ("bf16", 128, 257, 16, 2), ("bf16", 128, 258, 17, 2), ("bf16", 128, 1030, 32, 2), ("bf16", 128, 300, 33, 2),
         ("f32", 64, 17, 3, 2), ("f32", 128, 255, 64, 2), ("f32", 64, 512, 8, 2), ("f32", 64, 513, 8, 2)]


@pytest.mark.parametrize("dtype,d,n,k,B", CASES)
def test_rows_at_the_borders(oracle, dtype, d, n, k, B):
    g = torch.Generator().manual_seed(7000 + n + k)
    N, heads = n * B, 2
    Q = torch.randn((1, heads, N, d), generator=g).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    cent = torch.randn((1, heads, n, d), generator=g) * 0.2
    sh = moba.Shape(1, heads, N, d, B, k, 0, binding.BF16 if dtype == "bf16" else binding.F32, 0.0, 0, 0)
    idx, _ = moba.topk(sh, Q.cuda(), cent.cuda())
    got = idx.cpu().numpy().reshape(heads * N, k)
    Q64, C = Q.double().numpy()[0], cent.double().numpy()[0]
    rows = np.arange(heads * N, dtype=np.int64)[::1 if n < 600 else 7]
    ref, kth = oracle.topk(Q64, C, B, k, rows=rows)
    _, exempt = parity.routing_check(oracle, got[rows], ref, kth, Q64, C, B, rows=rows)
    assert exempt < 0.02
    assert (np.diff(np.where(got < 0, np.iinfo(np.int32).max, got), axis=-1) >= 0).all()


@pytest.mark.parametrize("d,n,k", [(64, 600, 8), (128, 300, 20), (64, 40, 20)])
def test_equal_scores_keep_the_lowest_blocks(d, n, k):
    B, N = 2, 2 * n
    g = torch.Generator().manual_seed(7)
    Q = torch.randn((1, 1, N, d), generator=g).to(torch.bfloat16).cuda()
    cent = torch.zeros((1, 1, n, d)).cuda()
    sh = moba.Shape(1, 1, N, d, B, k, 0, binding.BF16, 0.0, 0, 0)
    got = moba.topk(sh, Q, cent)[0].cpu().numpy()[0, 0]
    for t in range(0, N, 5):
        c = min(k, t // B)
        assert got[t].tolist() == list(range(c)) + [-1] * (k - c)
    # packed: a short sequence in front of one with many blocks, neither sees the other
    lens = [37, N - 37]
    lay = moba.VarlenLayout(np.array([0, 37, N]), B)
    Tp = lay.padded_tokens
    sh = moba.Shape(1, 1, Tp, d, B, k, 0, binding.BF16, 0.0, 0, 0)
    got = lay.unpad(moba.topk_varlen(sh, lay, lay.pad(Q), torch.zeros((1, 1, Tp // B, d)).cuda())[0])
    got = got.cpu().numpy()[0, 0]
    for t in range(0, N, 5):
        at, first = (t, 0) if t < lens[0] else (t - lens[0], 19)
        c = min(k, at // B)
        assert got[t].tolist() == list(range(first, first + c)) + [-1] * (k - c)


# the two sweeps take calls of many rows only: (d, blocks, k, B, heads, conv width), both sides of each rule
@pytest.mark.parametrize("d,n,k,B,heads,conv", [(64, 513, 8, 32, 19, 0), (64, 512, 8, 32, 19, 0), (64, 1025, 3, 32, 10, 0),
                                                (64, 513, 9, 32, 19, 0), (128, 448, 8, 32, 21, 0), (128, 447, 8, 32, 21, 0),
                                                (128, 500, 32, 32, 19, 4), (128, 500, 17, 32, 19, 3), (128, 500, 32, 32, 19, 0),
                                                (128, 2048, 32, 32, 5, 4), (128, 2048, 17, 32, 5, 3), (128, 2047, 24, 32, 5, 4)])
def test_two_sweeps_keep_what_the_exact_search_keeps(d, n, k, B, heads, conv):
    g = torch.Generator(device="cuda").manual_seed(n + k)
    N = n * B
    Q = torch.randn((1, heads, N, d), generator=g, device="cuda").to(torch.bfloat16)
    cent = torch.randn((1, heads, n, d), generator=g, device="cuda") * 0.2
    cent[:, -1] = 0.0                                # one head of equal scores: its strips are searched again
    got, want = (moba.topk(moba.Shape(1, heads, N, d, B, k, conv, binding.BF16, 0.0, flags, 0), Q, cent)[0]
                 for flags in (0, binding.FLAG_GATE_EXACT_SEARCH))
    # (both decide by the same three-term sums)
    assert torch.equal(got, want)


@pytest.mark.parametrize("d,k,heads,kv,lens", [(64, 8, 8, 2, [900, 33, 26000, 500, 12000]), (64, 1, 8, 4, [17000, 20000, 700]),
                                               (128, 3, 8, 1, [5, 21000, 18000]), (128, 8, 10, 0, [30000, 1200])])
def test_two_sweeps_on_packed_batches_and_shared_heads(d, k, heads, kv, lens):
    """Strips that begin in one sequence and end in another, strips of a long one with few candidates of a
    short one among them, centroids of a key/value head that several query heads share; the last of these has
    equal scores, so that its strips are searched again."""
    B = 32
    lay = moba.VarlenLayout(np.concatenate([[0], np.cumsum(lens)]), B)
    Tp, hkv = lay.padded_tokens, kv or heads
    assert heads * Tp >= 300000 and Tp // B > 512
    g = torch.Generator(device="cuda").manual_seed(d + k)
    Q = torch.randn((1, heads, Tp, d), generator=g, device="cuda").to(torch.bfloat16)
    cent = torch.randn((1, hkv, Tp // B, d), generator=g, device="cuda") * 0.2
    if hkv > 1:
        cent[:, -1] = 0.0
    shapes = [moba.Shape(1, heads, Tp, d, B, k, 0, binding.BF16, 0.0, flags, kv) for flags in (0, binding.FLAG_GATE_EXACT_SEARCH)]
    got, want = (moba.topk_varlen(sh, lay, Q, cent)[0] for sh in shapes)
    assert torch.equal(got, want)
    got, want = (moba.topk(sh, Q, cent)[0] for sh in shapes)             # the same as one sequence
    assert torch.equal(got, want)


@pytest.mark.parametrize("d,n,k,B,heads", [(64, 600, 8, 32, 16), (128, 450, 5, 32, 22)])
def test_two_sweeps_of_scores_closer_than_their_sums_can_tell(d, n, k, B, heads):
    """Queries and centroids of one sign with a common part: the scores are near |q| |c| and differ by about 2^-14 of
    it, so that every row has candidates inside the error of the two-term scores."""
    g = torch.Generator(device="cuda").manual_seed(n)
    N = n * B
    Q = (1.0 + 0.1 * torch.rand((1, heads, N, d), generator=g, device="cuda")).to(torch.bfloat16)
    cent = 1.0 + 2.0 ** -10 * torch.randn((1, heads, n, d), generator=g, device="cuda")
    got, want = (moba.topk(moba.Shape(1, heads, N, d, B, k, 0, binding.BF16, 0.0, flags, 0), Q, cent)[0]
                 for flags in (0, binding.FLAG_GATE_EXACT_SEARCH))
    assert torch.equal(got, want)


@pytest.mark.parametrize("d,n,k,heads,over", [(64, 1024, 8, 10, 3), (64, 1024, 8, 10, 16), (64, 1024, 2, 10, 100), (128, 1030, 8, 10, 16),
                                              (128, 2048, 32, 5, 3)])
def test_two_sweeps_of_neighbours_alike(d, n, k, heads, over):
    """Centroids smoothed over neighbouring blocks: a query's best blocks lie side by side, and near-equal ones
    send strips to the other search."""
    B = 32
    g = torch.Generator(device="cuda").manual_seed(n + over)
    Q = torch.randn((1, heads, n * B, d), generator=g, device="cuda").to(torch.bfloat16)
    window = torch.hann_window(2 * over + 1, device="cuda").view(1, 1, -1)
    cent = torch.randn((heads * d, 1, n), generator=g, device="cuda")
    cent = torch.nn.functional.conv1d(cent, 0.2 * window / window.norm(), padding=over).view(1, heads, d, n).transpose(2, 3).contiguous()
    got, want = (moba.topk(moba.Shape(1, heads, n * B, d, B, k, 4, binding.BF16, 0.0, flags, 0), Q, cent)[0]
                 for flags in (0, binding.FLAG_GATE_EXACT_SEARCH))
    assert torch.equal(got, want)


def test_zero_queries_in_strips_of_many_blocks():
    """A packed batch whose short sequences begin inside a strip that also sees a long one: their queries have
    one to three candidates, and with a query of zeros these are equal: the lowest blocks are kept."""
    lens, heads, d, B, k = [69968, 48, 53, 37, 9000], 4, 64, 16, 1
    offs = np.concatenate([[0], np.cumsum(lens)])
    lay = moba.VarlenLayout(offs, B)
    Tp = lay.padded_tokens
    g = torch.Generator(device="cuda").manual_seed(12)
    Q = torch.randn((1, heads, Tp, d), generator=g, device="cuda").to(torch.bfloat16)
    Q[:, :, 69968:lay.pad_offsets_host[4]] = 0.0
    cent = torch.randn((1, heads, Tp // B, d), generator=g, device="cuda") * 0.2
    got, want = (moba.topk_varlen(moba.Shape(1, heads, Tp, d, B, k, 0, binding.BF16, 0.0, flags, 0), lay, Q, cent)[0]
                 for flags in (0, binding.FLAG_GATE_EXACT_SEARCH))
    own = np.arange(48) // B
    first = 69968 // B
    assert got[0, 0, 69968:69968 + 48, 0].tolist() == [first if o > 0 else -1 for o in own]
    assert torch.equal(got, want)
