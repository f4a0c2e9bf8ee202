"""The list builder where a workgroup takes several chunks of queries (sparse routing of many slices): the same lists as slice by
slice, where it takes one; with and without places, one range of blocks and several, a last group and chunk that are not full."""
import pytest
import torch

import paper_2511_11571_amd as moba
from paper_2511_11571_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [0, binding.FLAG_REFERENCE_KERNELS])
@pytest.mark.parametrize("heads,N,B,k", [(64, 65536, 64, 2), (48, 65600, 64, 2), (40, 66016, 32, 3), (150, 16416, 32, 1), (36, 98400, 96, 2)])
def test_same_lists_as_slice_by_slice(heads, N, B, k, flags):
    g = torch.Generator(device="cuda").manual_seed(heads + N)
    own = (torch.arange(N, device="cuda") // B).view(1, 1, N, 1)
    e = torch.arange(k, device="cuda").view(1, 1, 1, k)
    start = torch.randint(0, 1 << 30, (1, heads, N, 1), generator=g, device="cuda")
    idx = (start + e * (own // k).clamp(min=1)) % own.clamp(min=1)             # k different past blocks, where there are k
    idx = torch.where(e < own, idx, -1).to(torch.int32).contiguous()
    shape = lambda h: moba.Shape(1, h, N, 64, B, k, 0, binding.BF16, 0.0, flags, 0)  # noqa: E731
    off, entries = moba.build_lists(shape(heads), idx)
    for h in range(0, heads, 5):
        o1, e1 = moba.build_lists(shape(1), idx[:, h:h + 1].contiguous())
        R = int(o1[0, 0, -1])
        assert torch.equal(off[0, h], o1[0, 0])
        assert R == int((idx[0, h] >= 0).sum()) and torch.equal(entries[0, h, :R], e1[0, 0, :R])
