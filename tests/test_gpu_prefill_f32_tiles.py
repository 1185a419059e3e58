"""fp32 prefill at the edges of its decomposition: query tiles of 16, 32 and 64 rows per workgroup, key tiles shared by
four wavefronts (fewer tiles than wavefronts, counts that do not divide), block sizes that are odd multiples of 16,
list rows beyond 64 entries, sequences that end inside a 16-key tile.  Bars: the task's 1e-5 (outputs) and 1e-3 (lse)."""
import numpy as np
import pytest
import torch

from oracle import powattn_oracle as orc
from paper_2503_03588_amd import binding as pa
from gpu_util import check_prefill, oracle_pattern

pytestmark = pytest.mark.gpu

CASES = [
    # hq, hkv, n, d, block, window, sink, flags
    (1, 1, 1, 64, 64, 1, 0, pa.POWER),           # one row, one key
    (1, 1, 17, 128, 16, 1, 0, pa.POWER),         # two query tiles, fewer key tiles than wavefronts
    (2, 1, 333, 64, 48, 2, 1, pa.POWER),         # block of three key tiles
    (2, 2, 401, 128, 80, 1, 1, pa.POWER),        # five
    (16, 2, 1041, 64, 64, 3, 1, pa.POWER),       # 64 queries per workgroup, ragged end
    (16, 4, 530, 128, 32, 2, 1, pa.POWER),       # 32 queries per workgroup
    (9, 3, 499, 64, 32, 2, 0, pa.POWER),         # too few tiles for more than 16 queries per workgroup
    (2, 1, 1100, 64, 16, 1, 0, pa.DENSE),        # implicit rows of up to 69 entries
    (1, 1, 1100, 128, 16, 69, 1, pa.POWER),      # listed rows of up to 69 entries
]


# query tiles of 16 rows per workgroup: as many as the registers hold while every compute unit gets a workgroup
@pytest.mark.parametrize("hq,hkv,n,d,block,tiles", [
    (2, 2, 1024, 64, 64, 1), (9, 3, 999, 64, 32, 2), (8, 2, 1041, 64, 64, 2), (8, 2, 2100, 64, 64, 4), (16, 4, 2100, 64, 48, 1),
    (2, 1, 1000, 128, 64, 1), (8, 2, 1100, 128, 64, 2), (8, 2, 2100, 128, 32, 2), (8, 2, 2100, 128, 16, 1),
])
def test_prefill_f32_every_form(hq, hkv, n, d, block, tiles):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    total, mq = -(-n // block) * (block // 16) * hq, 1
    while mq < 256 // d and block % (32 * mq) == 0 and total // (2 * mq) >= cus:
        mq *= 2
    assert mq == tiles
    check_prefill(pa.Pattern(block, 2, 1), 1, hq, hkv, n, d, "f32", 400 + n)


# few query tiles: the output's columns are dealt to two workgroups, or four at head_dim 128
@pytest.mark.parametrize("hq,hkv,n,d,block,parts", [
    (2, 2, 1024, 64, 64, 2), (1, 1, 2033, 64, 16, 2), (2, 1, 1041, 64, 64, 1),          # (272 tiles: one)
    (1, 1, 1000, 128, 16, 4), (3, 1, 300, 128, 48, 4), (2, 1, 1001, 128, 64, 2), (4, 2, 1100, 128, 64, 1),
])
def test_prefill_f32_columns_dealt_to_workgroups(hq, hkv, n, d, block, parts):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    tiles = -(-n // block) * (block // 16) * hq
    want = 4 if d == 128 and 4 * tiles <= cus else 2 if 2 * tiles <= cus else 1
    assert want == parts
    check_prefill(pa.Pattern(block, 2, 1), 1, hq, hkv, n, d, "f32", 500 + n)


@pytest.mark.parametrize("hq,hkv,n,d,block,window,sink,flags", CASES)
def test_prefill_f32_tiles(hq, hkv, n, d, block, window, sink, flags):
    check_prefill(pa.Pattern(block, window, sink, flags), 1, hq, hkv, n, d, "f32", 300 + n)


def test_prefill_f32_list_order_and_empty_row():
    """A caller's own list: the diagonal block first, entries to be passed over, and a row without any key."""
    pat = pa.Pattern(32, 1, 0)
    n, d = 96, 64
    q, k, v = (torch.randn((1, 1, n, d), generator=torch.Generator().manual_seed(7 + x)) for x in range(3))
    cnt = torch.tensor([2, 0, 3], dtype=torch.int32, device="cuda")
    idx = torch.tensor([[0, 1, -1], [0, 1, -1], [2, -1, 0]], dtype=torch.int32, device="cuda")
    o, lse = pa.prefill(pat, cnt, idx, q.cuda(), k.cuda(), v.cuda())
    o, lse = o.cpu().double()[0, 0], lse.cpu().double()[0, 0]
    s = (q.double() @ k.double().transpose(2, 3))[0, 0] / d ** 0.5
    t = torch.arange(n)
    blk = t // 32
    keep = (t[:, None] >= t[None]) & torch.tensor([[True, False, False], [False] * 3, [True, False, True]])[blk][:, blk]
    s = s.masked_fill(~keep, -float("inf"))
    rows = blk != 1
    ref = torch.softmax(s[rows], -1) @ v.double()[0, 0]
    assert float((o[rows] - ref).abs().max()) <= 1e-5
    assert float((lse[rows] - torch.logsumexp(s[rows], -1)).abs().max()) <= 1e-3
    assert float(o[~rows].abs().max()) == 0.0 and bool(torch.isneginf(lse[~rows]).all())


@pytest.mark.parametrize("at", [0, 383, 640])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("hq", [1, 16])                      # 16 and 64 queries to a workgroup
def test_prefill_f32_non_finite_keys_reach_the_rows_that_attend_them(hq, bad, at):
    """A key that is no number, or so large that its score is one of the infinities: the rows that softmax leaves without
    a result are the rows that have none here, whichever wavefront held the key (key 0: row 0 attends nothing else)."""
    pat = pa.Pattern(64, 2, 1)
    n, d = 641, 64
    gen = torch.Generator().manual_seed(11)
    q, k, v = (torch.randn((1, h, n, d), generator=gen) for h in (hq, 1, 1))
    k[0, 0, at, 3] = bad
    q[0, 0, -1, 3] = 1.0                                     # (the only row that attends key 640: its score is +inf)
    cnt, idx, _ = pa.mask_build(pat, n)
    o, lse = pa.prefill(pat, cnt, idx, q.cuda(), k.cuda(), v.cuda())
    o, lse = o.cpu().double()[0], lse.cpu().double()[0]
    keep = torch.from_numpy(orc.token_mask(n, oracle_pattern(pat)))
    s = (q[0].double() @ k[0, 0].double().T) / d ** 0.5
    s = s.masked_fill(~keep, -float("inf"))
    ref = torch.softmax(s, -1) @ v[0, 0].double()
    none = torch.isnan(ref).all(-1)
    assert int(none.sum()) > 0 and torch.equal(torch.isnan(o).all(-1), none) and torch.equal(torch.isnan(o).any(-1), none)
    assert bool(((o - ref).abs() <= 1e-5)[~none].all())
    assert bool(((lse - torch.logsumexp(s, -1)).abs() <= 1e-3)[~none].all())


@pytest.mark.parametrize("d,block,chains", [(64, 16, 4), (64, 32, 4), (64, 64, 2), (128, 16, 4), (128, 32, 4)])
def test_prefill_f32_scores_are_summed_in_short_chains(d, block, chains):
    """Sequences of one token: the log-sum-exp is the score.  Its error is that of an fp32 sum of d products, which grows
    with the length of the chain of additions: no further (root mean square, 15 % for 8192 draws and for the order
    inside a matrix instruction) from 64 bits than `chains` sums of every chains-th product (one chain: 1.5 .. 2 times)."""
    b, h = 64, 128                                           # 8192 rows: the form that the block size selects
    gen = torch.Generator().manual_seed(13)
    q, k, v = (torch.randn((b, h, 1, d), generator=gen) for _ in range(3))
    pat = pa.Pattern(block, 1, 0)
    cnt, idx, _ = pa.mask_build(pat, 1)
    _, lse = pa.prefill(pat, cnt, idx, q.cuda(), k.cuda(), v.cuda())
    qn, kn = (t.numpy().reshape(b * h, d) for t in (q, k))
    exact = (qn.astype(np.float64) * kn).sum(-1) / np.sqrt(d)

    def rms_of(n):
        sums = np.zeros((n, b * h), dtype=np.float32)
        for x in range(d):                                   # a float64 product of two floats is exact: a fused multiply-add
            sums[x % n] = (sums[x % n] + qn[:, x].astype(np.float64) * kn[:, x]).astype(np.float32)
        while len(sums) > 1:
            sums = sums[::2] + sums[1::2]
        m = sums[0] * np.float32(np.float32(1 / np.sqrt(d)) * np.float32(1.44269504))
        return float(np.sqrt(((m * np.float32(0.69314718) - exact) ** 2).mean()))
    got = float(np.sqrt(((lse.double().cpu().numpy().reshape(-1) - exact) ** 2).mean()))
    print(f"d {d} block {block}: {got:.3e}; 1 / 2 / 4 chains {rms_of(1):.3e} {rms_of(2):.3e} {rms_of(4):.3e}", flush=True)
    assert got <= 1.15 * rms_of(chains)
