"""The merge of cut items, by item and by range, against the oracle: many parts
per item, a handful, spans as few as waves, every row-tile count, both sides of
the rule that picks the layout (twice the items against the ranges)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_29364_amd as nsd
from workload import custom_config, make_meta, make_layer
from parity import i32, u16, check_attention

pytestmark = pytest.mark.gpu


def check_pool(meta, lay, kp, vp):
    """The pool after a fused pass: the arriving requests' blocks, every other byte as it was."""
    want = oracle.gather.kv_gather(u16(lay.k_stage)[None], u16(lay.v_stage)[None],
                                   u16(lay.k_pool)[None], u16(lay.v_pool)[None], meta.src_ids,
                                   meta.dst_ids)
    for got, ref in zip((kp, vp), want):
        assert np.array_equal(u16(got)[None], ref)

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
    kp, vp = lay.k_pool.clone(), lay.v_pool.clone()
    with nsd.attention_waves(waves):
        if fused:
            out = nsd.gather_verify_attention(
                lay.q, kp, vp, lay.k_stage, lay.v_stage, i32(meta.block_table, device),
                i32(meta.stage_table, device), *args)
        else:
            out = nsd.verify_attention(lay.q, kp, vp, i32(meta.block_table, device), *args)
    torch.cuda.synchronize()
    check_attention(meta, lay, out, range(bs))
    check_pool(meta, lay, kp, vp)


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
    check_pool(meta, lay, kp, vp)


COPY_MODE = [
    # (Hq, Hkv, D, K, waves, declared longest context or None): 64 of 1024 waves attend, the
    # others copy the staged blocks (their bytes per wave are below 0.4 of the attention's)
    (8, 2, 128, 3, 1024, None),
    (4, 2, 64, 4, 1024, None),
    (8, 2, 128, 3, None, 81920),     # the wave split by a long declared context
    (16, 2, 128, 7, None, 20480),    # 64 rows
]


@pytest.mark.parametrize("case", range(len(COPY_MODE)))
@pytest.mark.parametrize("arriving", ["some", "all"])
def test_copy_mode(device, case, arriving):
    hq, hkv, d, k, waves, declared = COPY_MODE[case]
    lens = [40, 300, 17, 129]
    cfg = custom_config(seed=970 + case, bs=4, num_q_heads=hq, num_kv_heads=hkv, head_dim=d,
                        vocab=0, n_arriving=0, pool_blocks=40, staging_order="shuffled")
    meta = make_meta(cfg, seq_lens=lens, depth=[k] * 4,
                     arriving=[True, arriving == "all", True, arriving == "all"])
    lay = make_layer(cfg, meta, 0, device)
    table, stage = meta.block_table, meta.stage_table
    if declared:
        pad = ((0, 0), (0, declared // 16 - table.shape[1]))
        table, stage = (np.pad(t, pad, constant_values=-1) for t in (table, stage))
    kp, vp = lay.k_pool.clone(), lay.v_pool.clone()
    with nsd.attention_waves(waves):
        out = nsd.gather_verify_attention(
            lay.q, kp, vp, lay.k_stage, lay.v_stage, i32(table, device), i32(stage, device),
            i32(meta.seq_lens, device), i32(meta.q_indptr, device), meta.max_q,
            declared or meta.max_seq_len)
    torch.cuda.synchronize()
    check_attention(meta, lay, out, range(4))
    check_pool(meta, lay, kp, vp)
