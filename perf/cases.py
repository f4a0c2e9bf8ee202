"""The work a user of this library has it do, as measurable cases.

Every case is one call chain through the public binding (``paper_2511_11571_amd``), with the tensors
resident on the GPU and the workspaces kept by the caller, as ``bench.py`` and the header describe:

  decode    a serving step: the last ``q_len`` positions of a sequence against a key/value cache and
            the cached block centroids
  forward   prefill or evaluation: (key conv +) centroids, gate + top-k + lists, forward attention
  train     the same followed by the backward at fixed routing (and the backward of the key conv)
  varlen    a training step over a packed batch of sequences of different lengths: copies into the
            padded layout, the step, copies of results and gradients back

Sizes are those of the benchmark configurations in ``workloads.py``, of the sweep, decode and
packed-batch modes of ``bench.py``, and odd relatives of them.
"""
import math

import torch

import paper_2511_11571_amd as moba
from paper_2511_11571_amd import binding

MOST_BLOCKS = 4096          # key blocks per head in drawn cases


def _case(kind, batch, heads, N, d, B, k, *, name=None, dtype="bf16", kv_heads=0, conv=0, skew=False, q_len=0,
          lens=""):
    c = {"kind": kind, "batch": batch, "heads": heads, "kv_heads": kv_heads, "N": N, "d": d, "B": B, "k": k,
         "dtype": dtype, "conv": conv, "skew": skew, "q_len": q_len, "lens": lens}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one token per sequence of a small batch against a long cache (ragged last block): the
        # smallest call, where latency and host work count
        _case("decode", 2, 16, 131109, 64, 128, 8, name="decode_1_of_131k", q_len=1),
        # a few tokens at once (speculative or chunked decoding), grouped-query heads, d = 128
        _case("decode", 1, 16, 32805, 128, 64, 32, name="decode_16_gqa_d128", kv_heads=4, q_len=16),
        # benchmark configuration 1: a small fp32 forward
        _case("forward", 1, 2, 2048, 64, 128, 3, name="forward_f32_2k", dtype="f32"),
        # fp32 forward and backward, as in checking a model's gradients at full precision
        _case("train", 2, 4, 4096, 64, 64, 7, name="train_f32_4k", dtype="f32"),
        # benchmark configuration 2: the forward of the shape the paper trains at
        _case("forward", 1, 16, 8192, 64, 128, 8, name="forward_8k_B128"),
        # odd sizes throughout: block count, heads and block size without powers of two
        _case("train", 3, 6, 10080, 64, 96, 10, name="train_10k_B96_odd"),
        # training with everything the paper adds: key conv, shared key/value heads, d = 128
        _case("train", 1, 16, 16384, 128, 64, 16, name="train_16k_gqa_conv_d128", kv_heads=4, conv=4),
        # benchmark configuration 5: hot blocks that most queries keep
        _case("train", 2, 16, 16384, 64, 64, 32, name="train_16k_skew", skew=True),
        # a packed batch of documents of very different lengths
        _case("varlen", 1, 16, 32768, 64, 32, 64, name="train_packed_32k",
              lens="9000,4097,12001,300,5000,2370"),
        # benchmark configuration 3: many small blocks, the headline workload
        _case("train", 1, 16, 32768, 64, 32, 64, name="train_32k_B32"),
        # benchmark configuration 4: long prefill with the key conv
        _case("forward", 1, 16, 131072, 128, 64, 32, name="prefill_131k_conv_d128", conv=4),
        # the far end of the paper's latency sweep, the largest
        _case("train", 2, 16, 524288, 64, 128, 8, name="train_524k_B128"),
    ]


def _spread(rng, lo, hi):
    """Log-uniform between lo and hi."""
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _routes(c):
    """(query, kept block) pairs in units of 64 channels and at most 128 keys."""
    return c["batch"] * c["heads"] * c["N"] * (c["k"] + 1) * (c["d"] / 64) * max(1.0, c["B"] / 128)


def draw(rng):
    most_routes = 0.8 * 32 * 524288 * 9
    while True:
        kind = rng.choice(["decode", "forward", "train", "train", "varlen", "f32"])
        d = rng.choice([64, 64, 128])
        heads = rng.choice([1, 2, 3, 4, 6, 8, 12, 16, 20, 32])
        kv = rng.choice([h for h in range(1, heads + 1) if heads % h == 0]) if rng.random() < 0.3 else 0
        if kind == "decode":
            B = rng.choice([32, 64, 100, 128, 256])
            N = int(_spread(rng, 2000, 262144))
            k = rng.randint(2, max(2, min(64, 4096 // B - 1)))
            batch = int(_spread(rng, 1, 32.99))
            c = _case(kind, batch, heads, N, d, B, k, kv_heads=kv, q_len=rng.choice([1, 1, 2, 3, 5, 8, 16]))
            cache = 4 * batch * (kv or heads) * N * d
            if N // B > MOST_BLOCKS or cache > 8e9:
                continue
            return c
        if kind == "f32":
            B = rng.choice([16, 32, 50, 64, 128])
            n = max(2, round(_spread(rng, 1024, 8192) / B))
            c = _case(rng.choice(["forward", "train"]), rng.choice([1, 2]), rng.choice([1, 2, 3, 4, 8]), n * B, d, B,
                      rng.randint(2, max(2, 1024 // B)), dtype="f32")
            return c
        B = rng.choice([32, 64, 96, 128, 256])
        k = rng.randint(2, max(2, min(64, rng.choice([1024, 2048, 4096]) // B - 1)))
        conv = rng.choice([0, 0, 3, 4])
        if kind == "varlen":
            lens = [int(_spread(rng, 100, 16000)) for _ in range(rng.randint(2, 12))]
            c = _case(kind, 1, heads, sum(lens), d, B, k, kv_heads=kv, conv=0, lens=",".join(map(str, lens)))
        else:
            n = max(4, round(_spread(rng, 1024, 524288) / B))
            skew = kv == 0 and rng.random() < 0.2
            c = _case(kind, rng.choice([1, 1, 2, 3]), heads, n * B, d, B, k, kv_heads=kv, conv=conv, skew=skew)
        n = c["N"] // B
        scores = c["batch"] * heads * c["N"] * n * (d / 64)
        if n > MOST_BLOCKS or _routes(c) > most_routes or scores > 0.5 * 32 * 524288 * 4096:
            continue
        return c


def _normal(g, shape, dtype):
    return torch.randn(shape, generator=g, dtype=torch.float32, device="cuda").to(dtype)


def prepare(case, seed):
    c = case
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    code = binding.BF16 if c["dtype"] == "bf16" else binding.F32
    b, h, hkv, N, d, B = c["batch"], c["heads"], c["kv_heads"] or c["heads"], c["N"], c["d"], c["B"]
    st = {"kind": c["kind"]}
    if c["kind"] == "decode":
        st["q_len"] = c["q_len"]
        st["Q"] = _normal(g, (b, h, c["q_len"], d), dt)
        st["K"], st["V"] = _normal(g, (b, hkv, N, d), dt), _normal(g, (b, hkv, N, d), dt)
        past = (N - 1) // B
        st["cent"] = st["K"][:, :, :past * B].reshape(b, hkv, past, B, d).mean(3, dtype=torch.float32).contiguous()
        st["shape"] = moba.Shape(b, h, N, d, B, c["k"], 0, code, 0.0, 0, c["kv_heads"])
        return st
    st["Q"] = _normal(g, (b, h, N, d), dt)
    st["K"], st["V"] = _normal(g, (b, hkv, N, d), dt), _normal(g, (b, hkv, N, d), dt)
    train = c["kind"] != "forward"
    if train:
        st["dO"] = _normal(g, (b, h, N, d), dt)
    st["conv_w"] = 0.5 * _normal(g, (hkv, d, c["conv"]), torch.float32) if c["conv"] else None
    if c["skew"]:
        # per head a direction u, |u| = 3, added to all keys of 1 % of the blocks; 0.5 u on every query
        u = _normal(g, (h, d), torch.float32)
        u = 3.0 * u / u.norm(dim=-1, keepdim=True)
        n = N // B
        order = torch.rand((b, h, n), generator=g, device="cuda").argsort(-1).argsort(-1)
        hot = (order < max(1, round(0.01 * n)))[..., None, None].float()
        K = st["K"].view(b, h, n, B, d)
        st["K"] = (K + hot * u[None, :, None, None, :]).to(dt).view(b, h, N, d)
        st["Q"] = (st["Q"] + 0.5 * u[None, :, None, :]).to(dt)
    if c["kind"] == "varlen":
        offs = [0]
        for x in c["lens"].split(","):
            offs.append(offs[-1] + int(x))
        st["layout"] = moba.VarlenLayout(offs, B)
        N = st["layout"].padded_tokens
    # a training program gives forward and backward one workspace, prepared once per step
    flags = binding.FLAG_SHARED_WORKSPACE if train else 0
    sh = moba.Shape(b, h, N, d, B, c["k"], c["conv"], code, 0.0, flags, c["kv_heads"])
    top, fwd, bwd = moba.workspace_bytes(sh)
    room = lambda n: torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")  # noqa: E731
    st["shape"], st["ws_topk"], st["ws"] = sh, room(top), room(max(fwd, bwd) if train else fwd)
    return st


def _step(st, Q, K, V, dO, top):
    sh = st["shape"]
    Ke, cent = moba.centroids(sh, K, st["conv_w"])
    idx, lists = top(Q, cent)
    O, lse = moba.forward(sh, Q, Ke, V, idx, lists, ws=st["ws"])
    out = {"idx": idx, "O": O, "lse": lse}
    if dO is not None:
        dQ, dK, dV = moba.backward(sh, Q, Ke, V, O, lse, dO, idx, lists, ws=st["ws"])
        if st["conv_w"] is not None:
            dK, out["dw"] = moba.key_conv_backward(sh, K, st["conv_w"], dK)
        out.update(dQ=dQ, dK=dK, dV=dV)
    return out


def run(state):
    st = state
    sh = st["shape"]
    if st["kind"] == "decode":
        O, lse, _ = moba.decode_forward(sh, st["q_len"], st["Q"], st["K"], st["V"], st["cent"], want_idx=False)
        return {"O": O, "lse": lse}
    if st["kind"] != "varlen":
        return _step(st, st["Q"], st["K"], st["V"], st.get("dO"),
                     lambda Q, cent: moba.topk(sh, Q, cent, ws=st["ws_topk"]))
    lay = st["layout"]
    Q, K, V, dO = (lay.pad(st[x]) for x in ("Q", "K", "V", "dO"))
    out = _step(st, Q, K, V, dO, lambda Q, cent: moba.topk_varlen(sh, lay, Q, cent, ws=st["ws_topk"]))
    del out["idx"]                       # names blocks of the padded layout
    return {name: lay.unpad(x) for name, x in out.items()}


def _counts(N, B, k):
    """Of one sequence of N tokens and one head: attended (query, key) pairs, kept past blocks and
    scored past blocks, summed over the queries."""
    n, r = divmod(N, B)
    kept = B * sum(min(j, k) for j in range(n)) + r * min(n, k)
    pairs = B * kept + n * B * (B + 1) // 2 + r * (r + 1) // 2
    return pairs, kept, B * (n * (n - 1) // 2) + r * n


def work(case):
    c = case
    b, h, hkv, N, d, B, k = (c["batch"], c["heads"], c["kv_heads"] or c["heads"], c["N"], c["d"], c["B"], c["k"])
    es = 2 if c["dtype"] == "bf16" else 4
    if c["kind"] == "decode":
        queries = b * h * c["q_len"]
        past = (N - 1) // B
        keys = min(k, past) * B + (N - 1) % B + 1
        # distinct rows only: the queries of a key/value head together cannot read more than its cache
        rows = b * hkv * min(N, keys * c["q_len"] * (h // hkv))
        return {"bytes": b * hkv * past * d * 4 + 2 * rows * d * es + queries * (2 * d * es + 4),
                "flops": queries * (2 * d * past + 4 * d * keys)}
    seqs = [int(x) for x in c["lens"].split(",")] if c["lens"] else [N]
    pairs, kept, scored = (b * h * sum(x) for x in zip(*(_counts(L, B, k) for L in seqs)))
    q_rows, kv_rows = b * h * N, b * hkv * N
    # Q, K, V read; O, lse, the routing and its lists written
    bytes_ = (2 * q_rows + 2 * kv_rows) * d * es + q_rows * (4 + 4 * k) + 4 * kept
    flops = 2 * d * scored + 4 * d * pairs
    if c["kind"] != "forward":
        bytes_ += (2 * q_rows + 2 * kv_rows) * d * es          # dO read; dQ, dK, dV written
        flops += 10 * d * pairs
    if c["conv"]:
        flops += (2 if c["kind"] == "forward" else 6) * c["conv"] * kv_rows * d
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    # "differ": kept blocks whose gate scores are closer than 32-bit sums can order
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3, "differ": 1e-3}
    # O and the gradients are stored in bf16 and P enters its products in bf16
    return {"rel": 1e-2, "max": 0.3, "differ": 1e-3}
