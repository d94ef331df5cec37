"""Verification over short caches (at most 256 positions): one work-group per
(sequence, KV head) combines its key groups and writes the rows itself.

Capacities around the 32-key tile, the four key groups and the 256-position
limit of this path (257 takes the split stream), sequences from empty over
shorter than the block to full, one to five 16-row blocks, both head sizes,
contiguous and paged, and a negative scale; tolerances as in
test_gpu_verify.py."""

import math

import numpy as np
import pytest

import oracle
from paper_2505_12728_amd import synth
from tests.gpu_util import assert_close, assert_lse_close
from tests.test_gpu_verify import run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap,k,hq,hkv,D,paged", [
    (1, 1, 2, 2, 128, False), (31, 4, 4, 2, 64, False), (32, 5, 8, 8, 128, False), (33, 6, 16, 4, 128, False),
    (64, 16, 2, 1, 64, False), (97, 7, 8, 2, 128, True), (128, 9, 16, 2, 128, False), (129, 4, 36, 4, 64, False),
    (160, 8, 8, 1, 64, True), (240, 7, 32, 8, 128, False), (255, 8, 16, 2, 128, False), (256, 5, 32, 4, 128, True),
    (257, 5, 32, 4, 128, False)])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_verify_short_cache(cap, k, hq, hkv, D, paged, sign):
    lens = np.array([cap, 0, min(cap, max(0, k - 2)), min(cap, 32), max(1, cap - 33), min(cap, 96)], np.int32)
    w = synth.Workload("short", "bf16", batch=len(lens), hq=hq, hkv=hkv, head_dim=D, kv_len=cap, block=k, paged=paged,
                       kv_len_min=1)
    d = synth.verify_inputs(w, seed=cap, kv_len=lens)
    scale = sign / math.sqrt(D)
    out, lse = run_gpu(d, scale=scale)
    ro, rl = oracle.verify_attention(d["q"].values, d["k_cache"].values, d["v_cache"].values, d["kv_len"], scale,
                                     page_table=d["page_table"])
    assert_close(out, ro, "bf16", "out")
    assert_lse_close(lse, rl, "bf16", "lse")


@pytest.mark.parametrize("kv,k,hq,hkv,D,B,paged", [
    (257, 5, 8, 8, 128, 1, False), (300, 16, 2, 2, 64, 3, True), (1201, 5, 32, 32, 128, 1, False),
    (2999, 4, 8, 2, 128, 2, True), (1500, 8, 4, 2, 64, 5, False),
    # a pair over 47 to 93 work-groups, more than one round of the merge
    (6001, 4, 4, 1, 128, 1, False), (6000, 16, 2, 2, 64, 2, True), (11999, 5, 3, 3, 128, 1, False),
    (9000, 8, 2, 1, 64, 5, True)])
def test_verify_one_row_block_few_tiles(kv, k, hq, hkv, D, B, paged):
    # at most 16 query rows per KV head and few tiles per work-group: two key
    # groups per work-group, ragged lengths with empty and very short ones
    lens = np.array([kv, 33, 0, max(1, k - 1), kv - 17][:B], np.int32)
    w = synth.Workload("few", "bf16", batch=B, hq=hq, hkv=hkv, head_dim=D, kv_len=kv, block=k, paged=paged,
                       kv_len_min=1)
    d = synth.verify_inputs(w, seed=kv, kv_len=lens)
    scale = 1.0 / math.sqrt(D)
    out, lse = run_gpu(d, scale=scale)
    ro, rl = oracle.verify_attention(d["q"].values, d["k_cache"].values, d["v_cache"].values, d["kv_len"], scale,
                                     page_table=d["page_table"])
    assert_close(out, ro, "bf16", "out")
    assert_lse_close(lse, rl, "bf16", "lse")


def test_verify_short_more_pairs_than_one_launch_holds():
    # 2^23 pairs of 17 rows are 2^32 threads at one work-group per pair: they
    # take the split stream.  One key per sequence, so every row is its head's
    # value row, exactly.
    import torch
    import paper_2505_12728_amd as sd
    B, hkv, g, D = 64, 1 << 17, 17, 64
    gen = torch.Generator(device="cuda").manual_seed(2)
    torch.cuda.empty_cache()
    q = torch.ones(B, 1, hkv * g, D, dtype=torch.bfloat16, device="cuda")
    kc = torch.ones(B, 1, hkv, D, dtype=torch.bfloat16, device="cuda")
    vc = torch.empty_like(kc)
    for b in range(B):
        vc[b] = torch.randn(1, hkv, D, generator=gen, device="cuda").bfloat16()
    kv = torch.ones(B, dtype=torch.int32, device="cuda")
    kv[5] = 0
    out, lse = sd.sd_verify_attention(q, kc, vc, kv, scale=0.125, lse=True)
    vc[5] = 0
    for b in range(B):
        assert torch.equal(out[b].view(hkv, g, D), vc[b, 0].float()[:, None].expand(hkv, g, D)), b
    want = torch.full((B,), 64 * 0.125, device="cuda")
    want[5] = float("-inf")
    assert torch.allclose(lse, want[:, None, None].expand_as(lse), rtol=1e-6)
    del q, kc, vc, out, lse
    torch.cuda.empty_cache()                    # 127 GB with the workspace
