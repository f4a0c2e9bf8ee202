"""Key-block lists from a given routing, at the edges between the one-launch builder of short slices and the
chunked one: every entry, its order and its place in the query's row, against a sort of the pairs on the CPU."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# (batch, heads, N, d, B, k): one block; ragged words; rows of a length that is no multiple of four; a
# workgroup of several blocks; the last shape inside each limit (LDS, entries) and the first one outside;
# slices of more than 512 and 1024 blocks
SHAPES = [
    (1, 1, 32, 64, 32, 1), (1, 1, 2 * 96, 64, 96, 1), (3, 1, 10 * 96, 64, 96, 5), (1, 2, 2048, 64, 128, 3),
    (2, 4, 4096, 64, 64, 7), (4, 16, 4096, 64, 128, 4), (1, 2, 8192, 64, 128, 4), (1, 2, 8192, 64, 128, 5),
    (1, 1, 8192, 128, 64, 3), (1, 3, 8192, 128, 64, 3), (5, 7, 3 * 1056, 64, 32, 9), (1, 16, 8192, 64, 128, 8),
    (1, 1, 32 * 600, 64, 32, 4), (1, 1, 32 * 1100, 64, 32, 3),
    # the chunked builder at the edges of its ranges of blocks, the last chunk of 256 queries whole and not
    # (and of the counts its fill pass adds up itself: 6084 and 6280, blocks that straddle threads' turns)
    (1, 2, 64 * 156, 64, 64, 5), (1, 2, 64 * 157, 64, 64, 5), (2, 3, 224 * 37, 64, 224, 6),
    # the most additions of all its workgroups together, 192 chunks x 32 blocks from 1344 and 1536 of them
    (1, 7, 1536 * 32, 64, 1536, 2), (1, 8, 1536 * 32, 64, 1536, 2),
    (1, 1, 64 * 512, 64, 64, 3), (1, 1, 64 * 513, 64, 64, 2), (1, 1, 32 * 1024, 64, 32, 5), (1, 1, 32 * 1025, 64, 32, 2),
]


def _routing(g, bh, N, B, k):
    """Ascending kept past blocks per query, -1 in the places left; some rows keep less than they could."""
    n = N // B
    own = np.arange(N) // B
    key = g.random((bh, N, n))
    key[:, np.arange(n)[None, :] >= own[:, None]] = 2.0
    kept = np.argsort(key, -1)[..., :k]
    if kept.shape[-1] < k:
        kept = np.concatenate([kept, np.full((bh, N, k - kept.shape[-1]), n)], -1)
    kept[kept >= own[None, :, None]] = n
    kept[g.random(kept.shape) < 0.1] = n
    kept = np.sort(kept, -1)
    kept[kept == n] = -1
    return kept.astype(np.int32)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_lists_of_a_routing(shape, dtype):
    import paper_2511_11571_amd as moba
    batch, heads, N, d, B, k = shape
    bh, n = batch * heads, N // B
    sh = moba.Shape(batch, heads, N, d, B, k, 0, moba.binding.BF16 if dtype == "bf16" else moba.binding.F32)
    # lists hold places where the attention kernels file partial results by them, which shows in the workspaces:
    # fp32 (every shape here), and bf16 where the automatic choice is the key-block-major one
    flagged = lambda flags: moba.workspace_bytes(moba.Shape(batch, heads, N, d, B, k, 0, sh.dtype, 0.0, flags))[1]
    with_places = dtype == "f32" or flagged(0) == flagged(moba.binding.FLAG_KEY_MAJOR) != flagged(moba.binding.FLAG_QUERY_TILES)
    idx = _routing(np.random.default_rng(N + k), bh, N, B, k)
    off, ql = moba.build_lists(sh, torch.from_numpy(idx).view(batch, heads, N, k).cuda())
    off, ql = off.cpu().numpy().reshape(bh, n + 1), ql.cpu().numpy().reshape(bh, -1)
    for s in range(bh):
        t, e = np.nonzero(idx[s] >= 0)
        j = idx[s][t, e]
        order = np.lexsort((t, j))
        want = np.concatenate([[0], np.cumsum(np.bincount(j, minlength=n))])
        assert (off[s] == want).all()
        got = ql[s, :want[-1]]
        assert ((got & 0xffffff) == t[order]).all()
        assert ((got >> 24) == (e[order] if with_places else 0)).all()
