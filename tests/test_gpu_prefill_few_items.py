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
