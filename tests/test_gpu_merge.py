"""The merge of cut items, by item and by range, against the oracle: many parts
per item, a handful, spans as few as waves, every row-tile count, both sides of
the rule that picks the layout (twice the items against the ranges)."""
import numpy as np
import pytest
import torch

import paper_2609_29364_amd as nsd
from workload import custom_config, make_meta, make_layer
from parity import i32, check_attention

pytestmark = pytest.mark.gpu

CASES = [
    # (Hq, Hkv, D, seq_lens, depths, waves)
    (8, 1, 128, [4099], [3], None),                      # one item, ~14 parts and up
    (8, 1, 64, [4099], [7], 1024),                       # 64 rows, one item
    (16, 2, 128, [130, 2049], [7, 0], 64),               # a short and a long item
    (4, 2, 64, [5, 90], [4, 4], 64),                     # fewer spans than waves
    (8, 8, 64, [700] * 8, [2] * 8, 128),                 # 64 items, 128 ranges: by item
    (8, 8, 64, [700] * 8, [2] * 8, 124),                 # 64 items, 124 ranges: by range
    (12, 4, 128, [4000] + [65] * 15, [4] * 16, 64),      # by range, one item of many parts
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("fused", [False, True])
def test_merge(device, case, fused):
    hq, hkv, d, lens, depth, waves = CASES[case]
    bs = len(lens)
    cfg = custom_config(seed=900 + case, bs=bs, num_q_heads=hq, num_kv_heads=hkv, head_dim=d,
                        vocab=0, n_arriving=0, pool_blocks=None)
    meta = make_meta(cfg, seq_lens=lens, depth=depth,
                     arriving=(np.arange(bs) % 2 == 0) & fused)
    lay = make_layer(cfg, meta, 0, device)
    args = (i32(meta.seq_lens, device), i32(meta.q_indptr, device), meta.max_q, meta.max_seq_len)
    with nsd.attention_waves(waves):
        if fused:
            out = nsd.gather_verify_attention(
                lay.q, lay.k_pool.clone(), lay.v_pool.clone(), lay.k_stage, lay.v_stage,
                i32(meta.block_table, device), i32(meta.stage_table, device), *args)
        else:
            out = nsd.verify_attention(lay.q, lay.k_pool, lay.v_pool,
                                       i32(meta.block_table, device), *args)
    torch.cuda.synchronize()
    check_attention(meta, lay, out, range(bs))


SKEWED = [
    # (Hq, Hkv, D, one long context, requests, rows K + 1)
    (4, 2, 64, 9000, 130, 5),        # by item: the long items hold ~256 parts, spans as few as waves
    (16, 1, 128, 5000, 200, 1),      # by item, one KV head
    (8, 2, 128, 9000, 300, 4),       # by range where waves are few (not fused)
    (8, 8, 64, 5000, 128, 2),        # 1024 items: by range, fused at the line too
]


@pytest.mark.parametrize("case", range(len(SKEWED)))
@pytest.mark.parametrize("fused", [False, True])
def test_merge_skewed(device, case, fused):
    """One context far longer than the others: its items hold most of the parts."""
    hq, hkv, d, longest, bs, rows = SKEWED[case]
    rng = np.random.default_rng(case)
    lens = rng.integers(16, 65, bs)
    lens[bs // 3] = longest
    cfg = custom_config(seed=950 + case, bs=bs, num_q_heads=hq, num_kv_heads=hkv, head_dim=d,
                        vocab=0, n_arriving=0, pool_blocks=None)
    meta = make_meta(cfg, seq_lens=lens, depth=np.full(bs, rows - 1),
                     arriving=(np.arange(bs) % 3 == 0) & fused)
    lay = make_layer(cfg, meta, 0, device)
    args = (i32(meta.seq_lens, device), i32(meta.q_indptr, device), meta.max_q, meta.max_seq_len)
    kp, vp = lay.k_pool.clone(), lay.v_pool.clone()
    if fused:
        out = nsd.gather_verify_attention(
            lay.q, kp, vp, lay.k_stage, lay.v_stage, i32(meta.block_table, device),
            i32(meta.stage_table, device), *args)
    else:
        out = nsd.verify_attention(lay.q, kp, vp, i32(meta.block_table, device), *args)
    torch.cuda.synchronize()
    check_attention(meta, lay, out, range(bs))
