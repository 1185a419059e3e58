"""Every check of the binding's arguments stands twice, in Python and in csrc/host.cpp.  Here each call, ordinary and then
altered in one place at a time, goes both ways over a stand-in for the library: the library must be called with the same
arguments, or not at all and with the same exception."""
import numpy as np
import pytest
import torch

from host_on_cpu import host_cpu, stand_in  # noqa: F401 (fixtures)
from paper_2503_03588_amd import binding as pa

PAT = pa.Pattern(64, 3, 1)
B, HQ, HKV, N, D = 2, 4, 2, 100, 64          # two blocks, the second a ragged one


def i32(*values):
    return torch.tensor(values, dtype=torch.int32)


def bf16(*shape):
    return torch.zeros(shape, dtype=torch.bfloat16)


def ordinary():
    """name -> arguments by name; the outputs are left to the call."""
    q, kv, pool = bf16(B, HQ, N, D), bf16(B, HKV, N, D), bf16(5, HKV, 64, D)
    lists = dict(kv_cnt=i32(1, 2), kv_idx=torch.zeros(2, 2, dtype=torch.int32))
    pages = dict(k_pages=pool, v_pages=pool.clone(), block_table=torch.zeros(B, 2, dtype=torch.int32))
    ws = torch.zeros(1 << 20, dtype=torch.uint8)
    piece = q[:, :, :30].contiguous()
    return {
        "prefill": dict(**lists, q=q, k=kv, v=kv.clone()),
        "prefill_chunk": dict(**lists, q=piece, k_cache=kv, v_cache=kv.clone(), q_start=40),
        "prefill_chunk_paged": dict(**lists, q=piece, **pages, q_start=40),
        "prefill_batch_paged": dict(**lists, q=piece, **pages, q_start=i32(40, 0), q_len=i32(30, 2)),
        "prefill_varlen": dict(**lists, q=q, k=kv, v=kv.clone(), seq_lens=i32(100, 3)),
        "decode": dict(q=bf16(B, HQ, D), k_cache=kv, v_cache=kv.clone(), kv_len=i32(100, 3), workspace=ws),
        "decode_paged": dict(q=bf16(B, HQ, D), **pages, kv_len=i32(100, 3), workspace=ws),
        "backward": dict(**lists, q=q, k=kv, v=kv.clone(), o=q.clone(), lse=torch.zeros(B, HQ, N), d_o=q.clone(), workspace=ws),
    }


class Sub(torch.Tensor):
    pass


def alterations(t):
    """One tensor argument, changed in one way; most of them are not what the call takes."""
    yield "fp32", t.float()
    yield "fp16", t.half()
    yield "int64", t.long()
    yield "a dimension less", t[0].contiguous()
    yield "a dimension more", t[None]
    for dim in range(t.dim()):
        if t.shape[dim] > 1:
            yield f"dimension {dim} shorter", t.narrow(dim, 0, t.shape[dim] - 1).contiguous()
            yield f"dimension {dim} not contiguous", torch.cat([t, t], dim).narrow(dim, 0, t.shape[dim])
    yield "empty", t[:0]
    yield "a subclass", t.as_subclass(Sub)
    yield "a parameter", torch.nn.Parameter(t, requires_grad=t.is_floating_point())
    yield "a negated view", torch._neg_view(t)
    yield "none", None
    yield "its address", t.data_ptr()
    yield "an array", t.float().numpy()


def cases():
    for name, args in ordinary().items():
        yield name, "as it is", args
        out = args["q"].clone()
        outs = {"dq": out, "dk": bf16(B, HKV, N, D), "dv": bf16(B, HKV, N, D)} if name == "backward" else {"o": out}
        yield name, "outputs given", {**args, **outs}
        if name != "backward":
            for lse in (torch.zeros(out.shape[:-1]), None):
                for want in (True, False, 1, 0, None):
                    yield name, f"lse {lse is not None}, want_lse {want!r}", {**args, "lse": lse, "want_lse": want}
        for scale in (0.25, 0, 1, -1.0, float("nan"), float("inf"), np.float64(0.5), np.float32(0.5), 1e300, "x", None):
            yield name, f"scale {scale!r}", {**args, "softmax_scale": scale}
        for pat in (pa.Pattern(128, 3, 1), pa.Pattern(64, 3, 1, pa.DENSE), pa.Pattern(-1, 3, 1), pa.Pattern(32, 3, 1, 7)):
            yield name, repr(pat), {**args, "pattern": pat}
        if "q_start" in args and not isinstance(args["q_start"], torch.Tensor):
            for q_start in (0, 98, 99, 1000, -1, 2 ** 40, 2 ** 70, np.int64(40), True, 40.0, i32(40)[0], None):
                yield name, f"q_start {q_start!r}", {**args, "q_start": q_start}
        if "workspace" in args:
            for ws in (None, args["workspace"][:8], args["workspace"].view(torch.int32), args["workspace"][::2]):
                yield name, f"workspace {ws if ws is None else tuple(ws.shape)}", {**args, "workspace": ws}
        if "kv_cnt" in args:
            yield name, "no lists", {**args, "kv_cnt": None, "kv_idx": None}
            yield name, "lists of one row", {**args, "kv_cnt": args["kv_cnt"][:1], "kv_idx": args["kv_idx"][:1]}
        for arg, t in {**args, **outs}.items():
            if isinstance(t, torch.Tensor):
                for how, changed in alterations(t):
                    if how == "its address" and arg not in ("q", "o"):
                        continue
                    yield name, f"{arg}: {how}", {**args, **({arg: outs[arg]} if arg in outs else {}), arg: changed}


def outcome(fake, name, args):
    """What the call did: the library's arguments (addresses of tensors that the call made itself are called "new"), or the
    type of the exception."""
    fake.seen.clear()
    args = dict(args)
    pattern = args.pop("pattern", PAT)
    try:
        result = getattr(pa, name)(pattern, **args)
    except Exception as e:
        assert not fake.seen
        return type(e).__name__
    (entry, values, passed), = fake.seen
    assert entry == "powattn_" + name
    tensors = [t for t in result if isinstance(t, torch.Tensor)]
    mine = {t.data_ptr() for t in tensors} - {t.data_ptr() for t in args.values() if isinstance(t, torch.Tensor)}
    shapes = [(tuple(t.shape), t.dtype) if isinstance(t, torch.Tensor) else t for t in result]
    if name == "backward" and args.get("workspace") is None or name.startswith("decode") and args.get("workspace") is None:
        mine.add(passed[-3])
    return values, tuple("new" if x in mine else "nan" if x != x else x for x in passed), shapes


@pytest.mark.parametrize("entry", sorted(ordinary()))
def test_both_ways_call_the_library_alike(stand_in, monkeypatch, entry):
    host, native = pa._native, 0
    for name, what, args in cases():
        if name != entry:
            continue
        monkeypatch.setattr(pa, "_native", host)
        with_native = outcome(stand_in, name, args)
        monkeypatch.setattr(pa, "_native", None)
        assert with_native == outcome(stand_in, name, args), (name, what)
        if what in ("as it is", "outputs given"):
            values = [args.get(k) for k in ARGUMENTS[name]]
            values = [{"softmax_scale": 0.0, "want_lse": True}.get(k, v) if v is None else v for k, v in zip(ARGUMENTS[name], values)]
            assert getattr(host, name)(PAT._values, *values) is not NotImplemented, what       # (these do go the native way)
            native += 1
    assert native == 2


LISTS, OUT = ["kv_cnt", "kv_idx"], ["o", "lse", "softmax_scale"]
ARGUMENTS = {
    "prefill": LISTS + ["q", "k", "v"] + OUT + ["want_lse"],
    "prefill_chunk": LISTS + ["q", "k_cache", "v_cache", "q_start"] + OUT + ["want_lse"],
    "prefill_chunk_paged": LISTS + ["q", "k_pages", "v_pages", "block_table", "q_start"] + OUT + ["want_lse"],
    "prefill_batch_paged": LISTS + ["q", "k_pages", "v_pages", "block_table", "q_start", "q_len"] + OUT + ["want_lse"],
    "prefill_varlen": LISTS + ["q", "k", "v", "seq_lens"] + OUT + ["want_lse"],
    "decode": ["q", "k_cache", "v_cache", "kv_len"] + OUT + ["workspace", "want_lse"],
    "decode_paged": ["q", "k_pages", "v_pages", "block_table", "kv_len"] + OUT + ["workspace", "want_lse"],
    "backward": LISTS + ["q", "k", "v", "o", "lse", "d_o", "dq", "dk", "dv", "softmax_scale", "workspace"],
}


def test_mask_build_both_ways(stand_in, host_cpu):
    for pattern in (PAT, pa.Pattern(64, 3, 1, pa.DENSE), pa.Pattern(-1, 3, 1), pa.Pattern(64, 0, 1, 0)):
        for n in (1, 64, 1000, 0, -5, 2 ** 40, 2 ** 70, 100.0, "x", np.int64(100)):
            stand_in.seen.clear()
            r = host_cpu.mask_build(pattern._values, n)
            native = [s for s in stand_in.seen]
            stand_in.seen.clear()
            try:
                want = pa.mask_build(pattern, n, device="cpu")       # (another device: always through Python)
            except Exception:
                assert r is NotImplemented and not native, (pattern, n)
                continue
            if r is NotImplemented:
                assert not native and type(n) is not int, (pattern, n)
                continue
            assert [t.shape for t in r[:2]] == [t.shape for t in want[:2]] and r[2] is None
            (e0, v0, a0), (e1, v1, a1) = native[0], stand_in.seen[0]
            assert (e0, v0, a0[0], a0[3:]) == (e1, v1, a1[0], a1[3:])
