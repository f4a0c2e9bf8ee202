"""Host-side behaviour of the C ABI: the library loads, exports every declared symbol,
and rejects bad arguments before anything is launched (so this runs without a GPU)."""
import ctypes
import os
import random
import re

import pytest

import paper_2511_11571_amd as moba
from paper_2511_11571_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(os.path.join(ROOT, "paper_2511_11571_amd", "libmoba.so")):
        from paper_2511_11571_amd import build
        build.build()
    return moba.lib()


def test_every_declared_symbol_is_exported(lib):
    header = open(os.path.join(ROOT, "include", "moba.h")).read()
    names = set(re.findall(r"\b(moba_[a-z_]+)\s*\(", header))
    assert {"moba_centroids", "moba_topk", "moba_forward", "moba_backward"} <= names
    for name in names:
        assert hasattr(lib, name), name


def _shape(**kw):
    base = dict(batch=1, heads=2, seqlen=1024, head_dim=64, block=32, topk=4)
    base.update(kw)
    return binding.Shape(**base)


def test_decode_forward_rejects_bad_arguments(lib):
    """Host-side checks only: every call returns before anything is launched."""
    one = ctypes.c_void_p(256)                 # never dereferenced on these paths
    sh = _shape(seqlen=1000).c()               # any length: the last block may be ragged
    f = lib.moba_decode_forward
    assert f(ctypes.byref(sh), 0, one, one, one, one, 31, one, one, None, None) == -1      # q_len
    assert f(ctypes.byref(sh), 1001, one, one, one, one, 31, one, one, None, None) == -1
    assert f(ctypes.byref(sh), 4, None, one, one, one, 31, one, one, None, None) == -1     # Q
    assert f(ctypes.byref(sh), 4, one, one, one, one, 30, one, one, None, None) == -1      # too few centroids
    assert f(ctypes.byref(sh), 4, one, one, one, None, 0, one, one, None, None) == -1
    big = _shape(seqlen=4098 * 32 + 5).c()     # more than 4096 complete blocks
    assert f(ctypes.byref(big), 1, one, one, one, one, 5000, one, one, None, None) == -2


def test_decode_workspace_counts_the_keys_there_are(lib):
    """Queries are shared by workgroups, which takes a workspace, from 512 KB of keys and values each: an own block that
    is hardly begun, or longer than the sequence, brings no more keys than it has."""
    def need(**kw):
        n = ctypes.c_size_t(99)
        assert lib.moba_decode_workspace(ctypes.byref(_shape(heads=1, **kw).c()), 1, ctypes.byref(n)) == 0
        return n.value
    assert need(seqlen=50, block=4096, topk=1) == 0
    assert need(seqlen=500, block=1 << 20, topk=8, head_dim=128) == 0
    assert need(seqlen=2047, block=4096, topk=1) == 0             # 512 KB less a row
    assert need(seqlen=2048, block=4096, topk=1) > 0
    assert need(seqlen=4096 + 7, block=4096, topk=1) > 0
    assert need(seqlen=(1 << 14) + 9, block=1 << 14, topk=0) == 0                # nine keys of the own block
    assert need(seqlen=(1 << 14) + 9000, block=1 << 14, topk=0) > 0


def test_decode_refuses_a_misaligned_workspace(lib):
    """The counters in it are counted up by 64-bit atomics.  (Host-side: nothing is launched.)"""
    one, sh = ctypes.c_void_p(256), _shape(heads=1, seqlen=4096 + 7, block=4096, topk=1).c()
    call = lambda ws, n: lib.moba_decode_forward_ws(ctypes.byref(sh), 1, one, one, one, one, 1, one, one, None, ctypes.c_void_p(ws), ctypes.c_size_t(n), None)  # noqa: E731
    assert call(256 + 4, 1 << 20) == -1 and call(256 + 1, 1 << 20) == -1
    assert call(256 + 4, 16) == -3                            # too small, as before


def _decode_shapes():
    rng = random.Random(5)
    for _ in range(4000):
        d, dtype = rng.choice([64, 128]), rng.choice([binding.F32, binding.BF16])
        block, topk = rng.choice([1, 16, 33, 64, 128, 1000, 4096]), rng.choice([0, 1, 3, 8, 16, 17, 40, 64, 300])
        seqlen = rng.choice([1, 50, 2047, 2048, 4096, 8193, 30000]) + rng.choice([0, 0, 1, 31])
        yield binding.Shape(rng.choice([1, 2, 5]), rng.choice([1, 4, 13, 32]), seqlen, d, block, topk, 0, dtype), rng.choice([1, 2, 3, 16])
    for es, d in ((2, 64), (2, 128), (4, 64), (4, 128)):          # at 512 KB, of a sequence and of kept blocks, and at 64 queries
        rows = (1 << 18) // (d * es)
        for seqlen, block, topk in ((rows, 4096, 1), (rows - 1, 4096, 1), (8191, 2, rows // 2), (8191, 2, rows // 2 - 1), (8192, 2, rows // 2 - 1)):
            for heads, q_len in ((1, 1), (64, 1), (65, 1), (8, 8), (3, 22)):
                yield binding.Shape(1, heads, seqlen, d, block, topk, 0, binding.BF16 if es == 2 else binding.F32), q_len


def test_decode_asks_for_a_workspace_where_there_can_be_one(lib, monkeypatch):
    """The binding's answer is the library's, for every shape, kept by no shape, and the library is not called where the
    answer is 0 by the rule's bounds: a decode step with a new shape is bound by the host."""
    asked = []
    binding._decode_workspace_bytes(_shape(heads=1, seqlen=9000, topk=255), 1)          # (looks the entry point up)
    real = binding._fn
    monkeypatch.setattr(binding, "_fn", lambda name, sig: asked.append(name) or real(name, sig))
    monkeypatch.setattr(binding, "lib", lambda: asked.append("lib") or lib)
    zero = shared = 0
    for sh, q_len in _decode_shapes():
        n = ctypes.c_size_t(99)
        if lib.moba_decode_workspace(ctypes.byref(sh.c()), q_len, ctypes.byref(n)) != 0:
            continue
        del asked[:]
        assert binding._decode_workspace_bytes(sh, q_len) == n.value, (sh, q_len)
        assert len(asked) <= 1
        shared += n.value > 0
        zero += not asked
    assert zero > 1000 and shared > 100
    # a step of a small model, a step against a long cache, many queries
    for sh, q_len in ((_shape(seqlen=700), 1), (_shape(heads=16, seqlen=131109, block=128, topk=8), 1),
                      (_shape(heads=16, batch=8, seqlen=30000, head_dim=128, block=64, topk=32), 1)):
        del asked[:]
        assert binding._decode_workspace_bytes(sh, q_len) == 0 and not asked


def test_grouped_query_shapes_are_accepted(lib):
    R = ctypes.c_int64(0)
    for kv in (0, 1, 2, 4):
        sh = _shape(heads=4, kv_heads=kv).c()
        assert lib.moba_routes_per_slice(ctypes.byref(sh), ctypes.byref(R)) == 0
    # sharing key/value heads shrinks the copies of K and V in the forward workspace
    assert moba.workspace_bytes(_shape(heads=4, kv_heads=1))[1] < moba.workspace_bytes(_shape(heads=4))[1]


@pytest.mark.parametrize("d", [64, 128])
def test_f32_backward_keeps_room_for_a_bounded_number_of_sums(lib, d):
    """fp32: a partial of dQ per (query, block) and part, (lse, -D) per query, D; with several shares of a walk, of which there are
    16 at most, fp32 dK and dV of every share."""
    several = 0
    for block, topk, n, heads in [(64, 0, 1, 1), (64, 0, 5, 3), (64, 7, 8, 1), (64, 8, 512, 2), (64, 2, 64, 40), (128, 3, 4096, 64),
                                  (4096, 0, 1, 1), (64, 1, 2, 4000), (256, 9, 30, 8)]:
        sh = _shape(heads=heads, seqlen=n * block, head_dim=d, block=block, topk=topk, dtype=binding.F32)
        rows, parts = heads * n * block, -(-block // 64)
        partials = 4 * d * rows * (topk + 1) * parts
        sums, rest = 8 * d * rows, 12 * rows + 1024
        if partials * (2 if d == 128 else 1) > 1 << 34:
            continue
        room = moba.workspace_bytes(sh)[2] - partials - rest
        assert -1024 <= room <= 16 * sums, (d, block, topk, n, heads)
        several += room >= 2 * sums - 1024
    assert several >= 4


def test_routes_and_workspace(lib):
    sh = _shape()
    n = 32
    assert moba.routes_per_slice(sh) == 32 * sum(min(c, 4) for c in range(n))
    assert moba.routes_per_slice(_shape(topk=0)) == 0
    assert moba.routes_per_slice(_shape(topk=1000)) == 32 * n * (n - 1) // 2
    a, b, c = moba.workspace_bytes(sh)
    assert a > 0 and b > 0 and c >= 4 * 2 * 1024


@pytest.mark.parametrize("kw,key_major", [
    (dict(heads=16, seqlen=32768, block=32, topk=64), False),                # headline shape: many kept blocks
    (dict(batch=2, heads=16, seqlen=16384, block=64, topk=32), False),       # skewed-routing shape
    (dict(heads=16, seqlen=8192, block=128, topk=8), True),                  # few kept blocks of many keys
    (dict(batch=2, heads=16, seqlen=524288, block=128, topk=8), True),       # the long end of the latency sweep
    (dict(heads=16, seqlen=131072, head_dim=128, block=64, topk=32, conv_width=4), True),
    (dict(heads=16, seqlen=16384, block=64, topk=60), False),                # dense routing: tiles
    (dict(heads=16, seqlen=8192, block=128, topk=0), False),                 # own block only
    # more than 4096 keys per query: too many for the fixed-point accumulators of the query tiles
    (dict(heads=2, seqlen=32768, block=32, topk=64), False),                 # 2080 keys: tiles
    (dict(heads=2, seqlen=32768, block=128, topk=64), True),                 # 8320 keys: key blocks
])
def test_default_cut_of_the_attention(kw, key_major):
    """With neither flag the library sizes (and runs) the forward and backward for the cut it
    estimates to be cheaper; seen from here through the workspace sizes, which differ."""
    kw = dict(dict(dtype=binding.BF16), **kw)
    forced = {f: moba.workspace_bytes(_shape(flags=f, **kw))[1:] for f in (binding.FLAG_KEY_MAJOR,
                                                                          binding.FLAG_QUERY_TILES)}
    picked = moba.workspace_bytes(_shape(**kw))[1:]
    if kw["topk"] > 0:
        assert forced[binding.FLAG_KEY_MAJOR] != forced[binding.FLAG_QUERY_TILES]
    assert picked == forced[binding.FLAG_KEY_MAJOR if key_major else binding.FLAG_QUERY_TILES]


@pytest.mark.parametrize("kw,status", [
    (dict(batch=0), -1), (dict(heads=-1), -1), (dict(seqlen=0), -1), (dict(block=0), -1),
    (dict(seqlen=1000), -1),            # not a multiple of the block
    (dict(topk=-1), -1), (dict(dtype=7), -1), (dict(conv_width=-2), -1), (dict(flags=32), -1),
    (dict(head_dim=96), -2), (dict(conv_width=9), -2), (dict(topk=5000), -2),
    (dict(seqlen=(1 << 24) + 32, topk=0), -2),      # longer than the 32-bit row offsets allow
    (dict(heads=6, kv_heads=4), -1),    # key/value heads must divide the query heads
    (dict(kv_heads=-1), -1), (dict(heads=2, kv_heads=4), -1),
])
def test_bad_shapes_are_rejected(lib, kw, status):
    sh = _shape(**kw).c()
    R = ctypes.c_int64(0)
    assert lib.moba_routes_per_slice(ctypes.byref(sh), ctypes.byref(R)) == status
    assert lib.moba_workspace_bytes(ctypes.byref(sh), None, None, None) == status
    assert lib.moba_strerror(status)


def test_null_pointers_and_short_workspace(lib):
    sh = _shape().c()
    z = ctypes.c_void_p(0)
    one = ctypes.c_void_p(256)          # never dereferenced: checks come first
    big = ctypes.c_size_t(1 << 40)
    assert lib.moba_routes_per_slice(None, None) == -1
    assert lib.moba_centroids(ctypes.byref(sh), z, z, z, one, z) == -1
    assert lib.moba_centroids(ctypes.byref(sh), one, one, z, one, z) == -1     # weights without conv
    conv = _shape(conv_width=4).c()
    assert lib.moba_centroids(ctypes.byref(conv), one, z, one, one, z) == -1   # conv without weights
    assert lib.moba_centroids(ctypes.byref(conv), one, one, z, one, z) == -1   # conv needs K_eff
    assert lib.moba_topk(ctypes.byref(sh), z, one, one, one, one, one, big, z) == -1
    assert lib.moba_topk(ctypes.byref(sh), one, one, one, z, one, one, big, z) == -1           # no blk_off
    assert lib.moba_topk(ctypes.byref(sh), one, one, one, one, one, z, big, z) == -3
    assert lib.moba_topk(ctypes.byref(sh), one, one, one, one, one, one, ctypes.c_size_t(8), z) == -3
    assert lib.moba_build_lists(ctypes.byref(sh), z, one, one, one, big, z) == -1
    assert lib.moba_forward(ctypes.byref(sh), one, one, one, one, one, one, z, one, one, big, z) == -1
    assert lib.moba_forward(ctypes.byref(sh), one, one, one, one, one, one, one, one, z, big, z) == -3
    assert lib.moba_backward(ctypes.byref(sh), one, one, one, one, one, one, one, one, one,
                             one, one, z, one, big, z) == -1
    assert lib.moba_backward(ctypes.byref(sh), one, one, one, one, one, one, one, one, one,
                             one, one, one, one, ctypes.c_size_t(16), z) == -3
    n = ctypes.c_size_t(0)
    assert lib.moba_key_conv_backward_workspace(ctypes.byref(sh), ctypes.byref(n)) == -1       # no conv
    assert lib.moba_key_conv_backward_workspace(ctypes.byref(conv), ctypes.byref(n)) == 0 and n.value > 0
    assert lib.moba_key_conv_backward(ctypes.byref(sh), one, one, one, one, one, one, big, z) == -1
    assert lib.moba_key_conv_backward(ctypes.byref(conv), one, one, z, one, one, one, big, z) == -1
    assert lib.moba_key_conv_backward(ctypes.byref(conv), one, one, one, one, one, one, big, z) == -1  # in place
    two = ctypes.c_void_p(512)
    assert lib.moba_key_conv_backward(ctypes.byref(conv), one, one, one, two, one, one, ctypes.c_size_t(8), z) == -3
    # key blocks per head: 16384 for the bf16 gate kernel, 4096 for the plain one (fp32 tensors,
    # or bf16 with the plain kernels asked for)
    for many in (_shape(seqlen=32 * 17000), _shape(seqlen=32 * 5000, dtype=binding.F32),
                 _shape(seqlen=32 * 5000, flags=binding.FLAG_REFERENCE_KERNELS)):
        assert lib.moba_topk(ctypes.byref(many.c()), one, one, one, one, one, one, big, z) == -2
        assert lib.moba_topk_static(ctypes.byref(many.c()), one, one, one, one, one, z) == -2


def test_binding_raises(lib):
    with pytest.raises(moba.MobaError):
        moba.routes_per_slice(_shape(head_dim=80))


def test_profile_session_misuse_is_rejected(lib):
    import ctypes
    ms = (ctypes.c_float * 4)()
    calls = (ctypes.c_int32 * 4)()
    assert lib.moba_profile_end(ms, calls) == -1            # no session open
    assert lib.moba_profile_begin() == 0
    assert lib.moba_profile_begin() == -1                   # already open
    assert lib.moba_profile_end(None, calls) == -1          # null array: the session stays open
    assert lib.moba_profile_end(ms, calls) == 0             # no launches: all zero, no HIP call
    assert list(calls) == [0, 0, 0, 0] and list(ms) == [0.0] * 4


def test_convolution_in_place_is_rejected(lib):
    one = ctypes.c_void_p(256)                 # never dereferenced on these paths
    sh = _shape(conv_width=4).c()
    assert lib.moba_centroids(ctypes.byref(sh), one, one, one, one, None) == -1      # K_eff == K
    sh1 = _shape(conv_width=0).c()
    assert lib.moba_centroids(ctypes.byref(sh1), None, None, None, one, None) == -1   # K missing


def test_threads_that_meet_on_a_new_shape_share_one_c_structure(monkeypatch):
    """Two threads make their first call with one Shape at the same time: the structure whose address either
    of them hands to C has to stay alive.  The first thread is held between finding no structure and storing
    its own until the second one has its address."""
    import threading
    sh = _shape()
    build, second_done = binding.Shape.c, threading.Event()
    first = threading.Thread(target=lambda: got.append(sh._ref()))

    def c(self):
        if threading.current_thread() is first:
            other = threading.Thread(target=lambda: (got.append(sh._ref()), second_done.set()))
            other.start()
            assert second_done.wait(10)
            other.join()
        return build(self)

    got = []
    monkeypatch.setattr(binding.Shape, "c", c)
    first.start()
    first.join()
    assert got == [ctypes.addressof(sh._cstruct)] * 2
