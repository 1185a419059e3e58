"""GPU parity: a launch of few work items runs workgroups of four wavefronts, a larger one of the same sequences eight.
Each wavefront computes the same 32 queries in the same order either way: the rows are bit-identical, and the oracle
holds for both.  Bar: 2e-2 on the outputs, 1e-3 on the log-sum-exp."""
import numpy as np
import pytest
import torch

from oracle import powattn_oracle as orc
from paper_2503_03588_amd import binding as pa
from paper_2503_03588_amd import synth
from gpu_util import TOL_LSE, TOL_O, oracle_pattern
from test_gpu_prefill_chunk_paged import pool_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,hq,hkv,d,n,many", [
    (64, 32, 8, 128, 1000, 3),      # 256 half-size items for one sequence: the last size with four wavefronts; 384 whole ones
    (64, 28, 4, 64, 600, 12),       # 14 tasks: the last half-size item of a block is half empty
    (128, 10, 2, 128, 700, 24),     # five heads a KV head: 20 tasks
    (256, 3, 1, 64, 513, 60),       # three query blocks, one query in the last
])
def test_same_rows_with_four_and_eight_wavefronts(B, hq, hkv, d, n, many):
    pat = pa.Pattern(B, 4, 1)
    q, k, v = synth.qkv(1, hq, hkv, n, d, "bf16", seed=79)
    cnt, idx, _ = pa.mask_build(pat, n)
    o1, l1 = pa.prefill(pat, cnt, idx, q.cuda(), k.cuda(), v.cuda())
    om, lm = pa.prefill(pat, cnt, idx, *(t.cuda().expand(many, -1, -1, -1).contiguous() for t in (q, k, v)))
    torch.cuda.synchronize()
    assert torch.equal(om, o1.expand_as(om)) and torch.equal(lm, l1.expand_as(lm))
    oo, olse = orc.attention(*(synth.to_numpy_storage(t) for t in (q, k, v)), oracle_pattern(pat))
    assert np.abs(o1.double().cpu().numpy() - oo).max() <= TOL_O["bf16"]
    assert np.abs(l1.double().cpu().numpy() - olse).max() <= TOL_LSE


@pytest.mark.parametrize("B,hq,hkv,d,q_start,q_len", [
    (64, 28, 4, 128, 33, 700),      # the first block holds one slice, the last one query
    (256, 7, 1, 64, 100, 150),      # one block only: slices 3 .. 7, no power of two of them
    (256, 12, 2, 128, 672, 450),    # first block: 3 slices, last one: 4, the second item of either half empty
    (128, 32, 8, 128, 127, 2),      # two blocks with one query each
])
def test_partial_blocks_take_fewer_items(B, hq, hkv, d, q_start, q_len):
    pat = pa.Pattern(B, 3, 1)
    n = q_start + q_len
    q, k, v = (t.cuda() for t in synth.qkv(5, hq, hkv, n, d, "bf16", seed=80))
    cnt, idx, _ = pa.mask_build(pat, n)
    want_o, want_l = pa.prefill(pat, cnt, idx, q, k, v)
    o, lse = pa.prefill_chunk(pat, cnt, idx, q[:, :, q_start:].contiguous(), k, v, q_start)
    torch.cuda.synchronize()
    assert torch.equal(o, want_o[:, :, q_start:]) and torch.equal(lse, want_l[:, :, q_start:])


def half_size_items(B, G, q_start, q_len):
    """Work items of one sequence and KV head in workgroups of four wavefronts (32 queries of one head each)."""
    items = 0
    for i in range(q_start // B, -(-(q_start + q_len) // B)):
        lo, hi = max(q_start, i * B), min(q_start + q_len, (i + 1) * B)
        items += -(-G * ((hi - 1) // 32 - lo // 32 + 1) // 4)
    return items


# What calls of ordinary size run: more half-size items than compute units, so workgroups of eight wavefronts, for every
# entry point and both head dimensions (the small shapes of the other files take four).  Sequence by sequence the launch
# is small enough for four, and the rows must be the same, bit for bit; the oracle holds for the last sequence.
MANY = [
    (64, 28, 4, 64, 5, 500, pa.POWER),            # 14 tasks a block: the second item has six
    (64, 28, 4, 128, 5, 500, pa.POWER),
    (128, 8, 2, 64, 14, 700, pa.POWER),           # two heads' four slices to an item
    (256, 6, 2, 128, 14, 700, 0),
    (192, 6, 2, 64, 16, 500, pa.POWER),           # a block size that is no power of two
    (64, 28, 4, 64, 5, 500, pa.DENSE),
    (128, 8, 2, 128, 14, 700, pa.DENSE),
]
KINDS = ["prompts", "chunk", "varlen", "paged", "batch_paged"]     # (the dense list has no paged form)


@pytest.mark.parametrize("kind,B,hq,hkv,d,batch,n,flags", [(kind, *m) for m in MANY for kind in KINDS[: 3 if m[-1] & pa.DENSE else 5]])
def test_many_items_take_eight_wavefronts(kind, B, hq, hkv, d, batch, n, flags):
    pat = pa.Pattern(B, 3, 1, flags)
    cus = torch.cuda.get_device_properties(0).multi_processor_count // 8 * 8
    a = 0 if kind in ("prompts", "varlen") else 97            # first query: three slices into a block of 64 or more
    assert hkv * half_size_items(B, hq // hkv, a, n - a) <= cus < batch * hkv * half_size_items(B, hq // hkv, a, n - a)
    q, k, v = synth.qkv(batch, hq, hkv, n, d, "bf16", seed=85)
    lists = (None, None) if flags & pa.DENSE else pa.mask_build(pat, -(-n // B) * B)[:2]
    qa = q[:, :, a:].contiguous().cuda()
    kp, vp, table = (t.cuda() for t in pool_for(k, v, [n] * batch, B, n_extra=2, seed=86))
    kg, vg = k.cuda(), v.cuda()
    starts = torch.full((batch,), a, dtype=torch.int32, device="cuda")
    lens = torch.full((batch,), n - a, dtype=torch.int32, device="cuda")

    def call(s):
        if kind == "prompts":
            return pa.prefill(pat, *lists, qa[s], kg[s], vg[s])
        if kind == "chunk":
            return pa.prefill_chunk(pat, *lists, qa[s], kg[s], vg[s], a)
        if kind == "paged":
            return pa.prefill_chunk_paged(pat, *lists, qa[s], kp, vp, table[s], a)
        if kind == "varlen":
            return pa.prefill_varlen(pat, *lists, qa[s], kg[s], vg[s], lens[s])
        return pa.prefill_batch_paged(pat, *lists, qa[s], kp, vp, table[s], starts[s], lens[s])

    o, lse = call(slice(None))
    for b in range(batch):
        o1, l1 = call(slice(b, b + 1))
        torch.cuda.synchronize()
        assert torch.equal(o[b:b + 1], o1) and torch.equal(lse[b:b + 1], l1), b
    oo, ol = orc.attention(*(synth.to_numpy_storage(t[-1:]) for t in (q, k, v)), oracle_pattern(pat))
    assert np.abs(o[-1:].double().cpu().numpy() - oo[:, :, a:]).max() <= TOL_O["bf16"]
    assert np.abs(lse[-1:].double().cpu().numpy() - ol[:, :, a:]).max() <= TOL_LSE


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,hkv,eight", [(4, 1, False), (28, 4, True)])      # 2 and 16 half-size items a block
def test_rows_too_long_to_be_chained(hq, hkv, eight, d):
    # more than 63 entries in a row: one workgroup to an item, of four or eight wavefronts; the window covers everything,
    # so the result is that of the dense list (in the larger case its persistent workgroups'); a padded batch gives the same rows
    n, B = 4200, 64
    cus = torch.cuda.get_device_properties(0).multi_processor_count // 8 * 8
    assert (hkv * half_size_items(B, hq // hkv, 0, n) > cus) == eight
    q, k, v = (t.cuda() for t in synth.qkv(1, hq, hkv, n, d, "bf16", seed=87))
    pat = pa.Pattern(B, 70, 0)
    cnt, idx, _ = pa.mask_build(pat, n)
    o, lse = pa.prefill(pat, cnt, idx, q, k, v)
    od, ld = pa.prefill(pa.Pattern(B, 1, 0, pa.DENSE), None, None, q, k, v)
    lens = torch.tensor([n - 777], dtype=torch.int32, device="cuda")
    ov, lv = pa.prefill_varlen(pat, cnt, idx, q, k, v, lens)
    torch.cuda.synchronize()
    assert idx.shape[1] > 63 and torch.equal(o, od) and torch.equal(lse, ld)
    assert torch.equal(ov[:, :, :n - 777], o[:, :, :n - 777]) and torch.equal(lv[:, :, :n - 777], lse[:, :, :n - 777])
    rows = np.unique(np.concatenate([[0, 63, 64, n - 1], np.random.default_rng(88).integers(0, n, 12)]))
    oo, ol = orc.attention_rows(*(synth.to_numpy_storage(t.cpu()) for t in (q, k, v)), rows, oracle_pattern(pat))
    assert np.abs(o[:, :, rows].double().cpu().numpy() - oo).max() <= TOL_O["bf16"]
    assert np.abs(lse[:, :, rows].double().cpu().numpy() - ol).max() <= TOL_LSE


# The same calls with more items than one and a half per compute unit (two where the device knows the lengths): the
# persistent variant, whose workgroups walk through several items.
@pytest.mark.parametrize("kind,B,hq,hkv,d,batch,n,flags", [(kind, *m[:4], 2 * m[4], *m[5:]) for m in MANY for kind in KINDS[: 3 if m[-1] & pa.DENSE else 5]])
def test_persistent_workgroups_give_the_same_rows(kind, B, hq, hkv, d, batch, n, flags):
    test_many_items_take_eight_wavefronts(kind, B, hq, hkv, d, batch, n, flags)


# Query blocks of at most four tasks: four wavefronts whatever the number of items, here more of them than two per compute unit,
# so their persistent variant, against the one-item variant of the one-sequence launches.
FOUR = [
    (64, 8, 8, 64, 12, 500, pa.POWER),            # two tasks a block
    (64, 8, 8, 128, 12, 500, pa.POWER),
    (64, 4, 2, 64, 40, 500, pa.POWER),            # four; two KV heads, whose items the XCDs share
    (64, 4, 2, 128, 40, 500, 0),
    (128, 8, 8, 128, 14, 700, pa.POWER),          # four slices of one head
    (64, 8, 8, 64, 12, 500, pa.DENSE),
    (128, 8, 8, 128, 14, 700, pa.DENSE),
]


@pytest.mark.parametrize("kind,B,hq,hkv,d,batch,n,flags", [(kind, *m) for m in FOUR for kind in KINDS[: 3 if m[-1] & pa.DENSE else 5]])
def test_persistent_workgroups_of_four_wavefronts(kind, B, hq, hkv, d, batch, n, flags):
    cus = torch.cuda.get_device_properties(0).multi_processor_count // 8 * 8
    a = 0 if kind in ("prompts", "varlen") else 97
    assert hq // hkv * B // 32 <= 4 and batch * hkv * half_size_items(B, hq // hkv, a, n - a) > 2 * cus
    test_many_items_take_eight_wavefronts(kind, B, hq, hkv, d, batch, n, flags)
