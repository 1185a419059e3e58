"""The work that programs built on this library have it do, as cases that can be timed.

`listed()` names the fixed cases, `draw()` gives more of the same ranges, `prepare()` makes what a program holds
before the call, `run()` is one pass through the public entry points, `work()` what a pass cannot do without and
`tolerance()` how far another correct implementation's results may lie.

A case's "kind" is the entry point it goes through:
  prefill      a whole prompt: powattn_mask_build and powattn_prefill (bf16 or fp32, sparse or the dense list)
  chunk        a piece of a prompt against the KV cache so far (contiguous or paged)
  varlen       a padded batch of prompts of different lengths, one launch
  batch_paged  the pieces of many sequences of a serving step, paged cache, one launch
  decode       one token for every sequence of a batch (contiguous or paged cache)
  train        forward and backward of one attention layer
"""
import math

import torch

from paper_2503_03588_amd import binding as pa


def _case(kind, name=None, **kw):
    c = {"kind": kind, "dtype": "bf16", "batch": 1, "hq": 32, "hkv": 8, "d": 128,
         "block": 64, "window": 4, "sink": 1, "dense": False, "paged": False}
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # The tiny full-precision configuration: what a numerics check or a small research model runs, and the
        # smallest prefill of all.
        _case("prefill", "prefill_f32_1k", dtype="f32", hq=2, hkv=2, d=64, n=1024, window=2),
        # A short prompt of odd length (a chat turn): few query blocks, latency counts.
        _case("prefill", "prefill_short", n=1000),
        # One layer over an ordinary long prompt.
        _case("prefill", "prefill_32k", n=32768),
        # The long-context prompt the method is for.
        _case("prefill", "prefill_128k", n=131072, block=128),
        # Chunked prefill of a long prompt: a piece that starts inside a block, against the pages written so far.
        _case("chunk", "chunk_2k_at_30k", hq=28, hkv=4, q_start=30001, q_len=2000, paged=True),
        # Prompts of mixed lengths that arrived together.
        _case("varlen", "varlen_batch32", batch=32, n_lo=300, n_hi=8192),
        # A serving step's prefill work: pieces of many sequences with different contexts so far.
        _case("batch_paged", "serving_step_32", batch=32, ctx_lo=0, ctx_hi=63000, q_lo=1, q_hi=2048),
        # Generation for one user: the smallest call there is.
        _case("decode", "decode_b1", len_lo=32001, len_hi=32001),
        # Generation for a small batch with long contexts, contiguous caches.
        _case("decode", "decode_b16_64k", batch=16, len_lo=65536, len_hi=65536),
        # Generation for a large serving batch of mixed contexts, paged cache.
        _case("decode", "decode_paged_b128", batch=128, len_lo=1000, len_hi=16384, paged=True),
        # A training step's attention in the paper's own setting (blocks of 256 keys, window of 5, one sink).
        _case("train", "train_32k_b256", hq=28, hkv=4, n=32768, block=256, window=5),
        # ... and at 128K, the longest gradient pass.
        _case("train", "train_128k", n=131072, block=128),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["prefill", "prefill", "prefill_f32", "chunk", "varlen", "batch_paged", "decode", "decode", "train", "train"])
    hq, hkv = rng.choice([(32, 8), (32, 8), (28, 4), (8, 8), (16, 2)])
    d = rng.choice([128, 128, 64])
    block = rng.choice([64, 64, 128, 256])
    window, sink = rng.choice([(4, 1), (4, 1), (5, 1), (4, 0), (2, 1), (9, 2)])
    kw = dict(hq=hq, hkv=hkv, d=d, block=block, window=window, sink=sink)
    if kind == "prefill":
        dense = rng.random() < 0.2
        return _case("prefill", n=_log_int(rng, 100, 24000 if dense else 131072), dense=dense, **kw)
    if kind == "prefill_f32":
        kw.update(hq=rng.choice([2, 4, 8]), hkv=2, block=rng.choice([16, 32, 64, 128]))
        return _case("prefill", dtype="f32", n=_log_int(rng, 64, 8192), **kw)
    if kind == "chunk":
        return _case("chunk", q_start=_log_int(rng, 100, 100000), q_len=_log_int(rng, 64, 8192), paged=rng.random() < 0.5, **kw)
    if kind == "varlen":
        n_hi = _log_int(rng, 256, 8192)
        return _case("varlen", batch=rng.choice([2, 5, 8, 16, 32]), n_lo=max(1, n_hi // rng.choice([2, 8, 27])), n_hi=n_hi, **kw)
    if kind == "batch_paged":
        return _case("batch_paged", batch=rng.choice([3, 8, 16, 32]), ctx_lo=0, ctx_hi=_log_int(rng, 1000, 63000),
                     q_lo=1, q_hi=_log_int(rng, 32, 2048), **kw)
    if kind == "decode":
        batch = rng.choice([1, 2, 4, 8, 16, 24, 32, 64, 128])
        len_hi = _log_int(rng, 300, 131072 if batch <= 8 else 65536 if batch <= 24 else 16384)
        return _case("decode", batch=batch, len_lo=max(1, len_hi // rng.choice([1, 2, 16])), len_hi=len_hi, paged=rng.random() < 0.5, **kw)
    return _case("train", n=_log_int(rng, 256, 65536), **kw)


# ---- what the cases have in common ---------------------------------------------------------------------------
def _pattern(case):
    flags = pa.DENSE | pa.POWER if case["dense"] else pa.POWER
    return pa.Pattern(case["block"], case["window"], case["sink"], flags)


def _spread(lo, hi, count):
    """`count` whole numbers spread evenly over lo .. hi, both ends among them."""
    if count == 1:
        return [hi]
    return [lo + (hi - lo) * k // (count - 1) for k in range(count)]


def _pieces(case):
    """(context so far, new rows) of every sequence of a serving step; long contexts do not always go with long pieces."""
    n = case["batch"]
    ctx, new = _spread(case["ctx_lo"], case["ctx_hi"], n), _spread(case["q_lo"], case["q_hi"], n)
    return [(ctx[k], new[(7 * k + 3) % n]) for k in range(n)]


def _lists(pat, n):
    if pat.flags & pa.DENSE:
        return None, None
    cnt, idx, _ = pa.mask_build(pat, n)
    return cnt, idx


def _page_table(gen, batch, blocks, spare):
    """Every block of every sequence on a page of its own, the pages in random order."""
    n_pages = batch * blocks + spare
    perm = torch.randperm(n_pages, generator=gen, device="cuda", dtype=torch.int32)
    return perm[: batch * blocks].reshape(batch, blocks).contiguous(), n_pages


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    b, hq, hkv, d, blk = (case[k] for k in ("batch", "hq", "hkv", "d", "block"))
    pat = _pattern(case)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=dt)

    def shuffled(values):
        order = torch.randperm(len(values), generator=gen, device="cuda")
        return torch.tensor(values, dtype=torch.int32, device="cuda")[order].contiguous()

    s = {"case": case, "pat": pat}
    kind = case["kind"]
    if kind in ("prefill", "train"):
        n = case["n"]
        s["q"], s["k"], s["v"] = normal(b, hq, n, d), normal(b, hkv, n, d), normal(b, hkv, n, d)
        if kind == "train":
            s["lists"] = _lists(pat, n)          # the same for every layer and step
            s["do"] = normal(b, hq, n, d)
        else:
            s["o"] = torch.empty_like(s["q"])
            s["lse"] = torch.empty((b, hq, n), dtype=torch.float32, device="cuda")
    elif kind == "chunk":
        total = case["q_start"] + case["q_len"]
        s["q"] = normal(b, hq, case["q_len"], d)
        s["o"] = torch.empty_like(s["q"])
        s["lse"] = torch.empty(s["q"].shape[:3], dtype=torch.float32, device="cuda")
        s["lists"] = _lists(pat, total)          # built once for the longest context; rows do not depend on the length
        if case["paged"]:
            s["table"], n_pages = _page_table(gen, b, -(-total // blk), 5)
            s["k"], s["v"] = normal(n_pages, hkv, blk, d), normal(n_pages, hkv, blk, d)
        else:
            s["k"], s["v"] = normal(b, hkv, total + 100, d), normal(b, hkv, total + 100, d)
    elif kind == "varlen":
        n = case["n_hi"]
        s["q"], s["k"], s["v"] = normal(b, hq, n, d), normal(b, hkv, n, d), normal(b, hkv, n, d)
        s["o"], s["lse"] = torch.zeros_like(s["q"]), torch.zeros((b, hq, n), dtype=torch.float32, device="cuda")
        s["lens"] = shuffled(_spread(case["n_lo"], n, b))
        s["lists"] = _lists(pat, n)
    elif kind == "batch_paged":
        pieces = _pieces(case)
        rows = max(r for _, r in pieces)
        order = torch.randperm(b, generator=gen, device="cuda")
        s["start"] = torch.tensor([c for c, _ in pieces], dtype=torch.int32, device="cuda")[order].contiguous()
        s["rows"] = torch.tensor([r for _, r in pieces], dtype=torch.int32, device="cuda")[order].contiguous()
        blocks = -(-max(c + r for c, r in pieces) // blk)
        blocks = max(blocks, -(-rows // blk))
        s["table"], n_pages = _page_table(gen, b, blocks, 5)
        s["q"] = normal(b, hq, rows, d)
        s["k"], s["v"] = normal(n_pages, hkv, blk, d), normal(n_pages, hkv, blk, d)
        s["o"], s["lse"] = torch.zeros_like(s["q"]), torch.zeros((b, hq, rows), dtype=torch.float32, device="cuda")
        s["lists"] = _lists(pat, blocks * blk)
    else:
        lens = _spread(case["len_lo"], case["len_hi"], b)
        s["lens"] = shuffled(lens)
        s["q"] = normal(b, hq, d)
        s["o"], s["lse"] = torch.empty_like(s["q"]), torch.empty((b, hq), dtype=torch.float32, device="cuda")
        cap = (-(-max(lens) // blk) + 1) * blk   # room for the tokens to come
        if case["paged"]:
            s["table"], n_pages = _page_table(gen, b, cap // blk, 5)
            s["k"], s["v"] = normal(n_pages, hkv, blk, d), normal(n_pages, hkv, blk, d)
        else:
            s["k"], s["v"] = normal(b, hkv, cap, d), normal(b, hkv, cap, d)
        s["ws"] = pa.decode_workspace(pat, b, hq, hkv, d, cap)
    return s


def run(s):
    case, pat = s["case"], s["pat"]
    kind = case["kind"]
    if kind == "prefill":
        cnt, idx = _lists(pat, case["n"])
        o, lse = pa.prefill(pat, cnt, idx, s["q"], s["k"], s["v"], o=s["o"], lse=s["lse"])
        return {"o": o, "lse": lse} if cnt is None else {"cnt": cnt, "idx": idx, "o": o, "lse": lse}
    if kind == "train":
        cnt, idx = s["lists"]
        o, lse = pa.prefill(pat, cnt, idx, s["q"], s["k"], s["v"])
        dq, dk, dv = pa.backward(pat, cnt, idx, s["q"], s["k"], s["v"], o, lse, s["do"])
        return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    if kind == "chunk":
        cnt, idx = s["lists"]
        if case["paged"]:
            return pa.prefill_chunk_paged(pat, cnt, idx, s["q"], s["k"], s["v"], s["table"], case["q_start"], o=s["o"], lse=s["lse"])
        return pa.prefill_chunk(pat, cnt, idx, s["q"], s["k"], s["v"], case["q_start"], o=s["o"], lse=s["lse"])
    if kind == "varlen":
        cnt, idx = s["lists"]
        return pa.prefill_varlen(pat, cnt, idx, s["q"], s["k"], s["v"], s["lens"], o=s["o"], lse=s["lse"])
    if kind == "batch_paged":
        cnt, idx = s["lists"]
        return pa.prefill_batch_paged(pat, cnt, idx, s["q"], s["k"], s["v"], s["table"], s["start"], s["rows"], o=s["o"], lse=s["lse"])
    if case["paged"]:
        return pa.decode_paged(pat, s["q"], s["k"], s["v"], s["table"], s["lens"], o=s["o"], lse=s["lse"], workspace=s["ws"])
    return pa.decode(pat, s["q"], s["k"], s["v"], s["lens"], o=s["o"], lse=s["lse"], workspace=s["ws"])


# ---- the work of a pass ----------------------------------------------------------------------------------------
def _row(case, i):
    """The key blocks that query block i attends: i-j < W, i-j zero or a power of two, or j < S (all j <= i when dense)."""
    if case["dense"]:
        return range(i + 1)
    row = set(range(max(0, i - case["window"] + 1), i + 1)) | set(range(min(case["sink"], i + 1))) | {i}
    p = 1
    while p <= i:
        row.add(i - p)
        p *= 2
    return row


def _row_len(case, i):
    if case["dense"]:
        return i + 1
    return len(_row(case, i))


def _pairs(case, start, stop):
    """Attended (query, key) pairs of the queries start .. stop-1 of one sequence."""
    blk, pairs = case["block"], 0
    for i in range(start // blk, -(-stop // blk)):
        lo, hi = max(start, i * blk), min(stop, (i + 1) * blk)
        pairs += (hi - lo) * (_row_len(case, i) - 1) * blk        # the blocks before the diagonal one, in full
        pairs += sum(range(lo - i * blk + 1, hi - i * blk + 1))   # the diagonal block, causal
    return pairs


def _keys(case, start, stop):
    """Keys that any of the queries start .. stop-1 attends."""
    blk, seen = case["block"], set()
    for i in range(start // blk, -(-stop // blk)):
        seen.update(_row(case, i))
    last = -(-stop // blk) - 1
    return sum(stop - j * blk if j == last else blk for j in seen)


def work(case):
    b, hq, hkv, d = case["batch"], case["hq"], case["hkv"], case["d"]
    size = 2 if case["dtype"] == "bf16" else 4
    kind = case["kind"]
    if kind in ("prefill", "train"):
        spans = [(0, case["n"])] * b
    elif kind == "chunk":
        spans = [(case["q_start"], case["q_start"] + case["q_len"])] * b
    elif kind == "varlen":
        spans = [(0, n) for n in _spread(case["n_lo"], case["n_hi"], b)]
    elif kind == "batch_paged":
        spans = [(c, c + r) for c, r in _pieces(case)]
    else:
        spans = [(n - 1, n) for n in _spread(case["len_lo"], case["len_hi"], b)]
    rows = sum(stop - start for start, stop in spans)
    pairs = sum(_pairs(case, *s) for s in spans)
    keys = rows if kind in ("prefill", "train", "varlen") else sum(_keys(case, *s) for s in spans)
    q_bytes, kv_bytes, lse_bytes = rows * hq * d * size, 2 * keys * hkv * d * size, rows * hq * 4
    fwd = {"bytes": 2 * q_bytes + kv_bytes + lse_bytes, "flops": 4 * d * hq * pairs}
    if kind != "train":
        return fwd
    # backward: q, k, v, o, lse, dO in, dq, dk, dv out; five products where the forward pass has two
    return {"bytes": fwd["bytes"] + 4 * q_bytes + 2 * kv_bytes + lse_bytes, "flops": fwd["flops"] + 10 * d * hq * pairs}


def tolerance(case):
    # About four times what these paths measure against the same attention in 64 bits (N = 1024 .. 4096):
    # fp32 rel 4.6e-7, max 3.6e-6; bf16 outputs rel 2.3e-3, max 2.8e-2 (one rounding to bf16 on top of that of the
    # probabilities); bf16 gradients rel 2.4e-3, max 5.5e-2, where max grows with the number of values drawn.
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 2e-5}
    if case["kind"] == "train":
        return {"rel": 1e-2, "max": 0.3}
    return {"rel": 1e-2, "max": 0.15}
