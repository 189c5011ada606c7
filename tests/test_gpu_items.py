"""The short-context attention (a workgroup per request, KV head and chunk)
against the oracle: every row-tile count at both head dims, contexts at the
edges of its spans (32 tokens), waves (128 tokens a step) and chunks, batches
whose longest request is cut while the others are whole, and a declared
longest context far beyond the real ones."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_29364_amd as nsd
from workload import custom_config, make_meta, make_layer
from parity import i32, u16, check_attention

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 16, 31, 32, 33, 96, 97, 127, 128, 129, 255, 257, 500]

CASES = [
    # (Hq, Hkv, D, seq_lens, depth, declared longest context or None)
    (2, 2, 64, EDGES, 0, None),                 # 1 row
    (8, 1, 64, EDGES, 7, None),                 # 64 rows
    (8, 2, 128, EDGES, 3, None),                # 16 rows
    (8, 2, 128, EDGES, 4, None),                # 20 rows
    (8, 2, 128, EDGES, 8, None),                # 36 rows: Q in LDS
    (16, 2, 128, EDGES, 7, None),               # 64 rows: one wave per SIMD
    (8, 2, 128, [1, 1024, 1025, 5000, 64], 4, None),          # above 512 KiB an item is cut
    (8, 2, 128, [1, 1024, 1025, 5000, 64], 8, None),
    (16, 2, 128, [3000, 70], 7, None),
    (4, 2, 64, [2048, 2049, 127, 9000], 4, None),
    (1, 1, 128, [1100] + [40] * 99, 0, None),                 # one request cut, 100 requests
    (8, 2, 128, [130, 40, 256, 9], 4, 4000),                  # cut by declaration only
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("fused", [False, True])
def test_items(device, case, fused):
    hq, hkv, d, lens, k, declared = CASES[case]
    bs = len(lens)
    depth = np.minimum(k, np.asarray(lens) - 1)
    cfg = custom_config(seed=700 + case, bs=bs, num_q_heads=hq, num_kv_heads=hkv, head_dim=d,
                        vocab=0, n_arriving=0, pool_blocks=None, staging_order="shuffled")
    meta = make_meta(cfg, seq_lens=lens, depth=depth,
                     arriving=(np.arange(bs) % 3 != 1) & fused)
    lay = make_layer(cfg, meta, 0, device)
    kp, vp = lay.k_pool.clone(), lay.v_pool.clone()
    table, stage = meta.block_table, meta.stage_table
    if declared:
        pad = ((0, 0), (0, -(-declared // 16) - table.shape[1]))
        table, stage = (np.pad(t, pad, constant_values=-1) for t in (table, stage))
    args = (i32(meta.seq_lens, device), i32(meta.q_indptr, device), meta.max_q,
            declared or meta.max_seq_len)
    if fused:
        out = nsd.gather_verify_attention(lay.q, kp, vp, lay.k_stage, lay.v_stage,
                                          i32(table, device), i32(stage, device), *args)
    else:
        out = nsd.verify_attention(lay.q, kp, vp, i32(table, device), *args)
    torch.cuda.synchronize()
    check_attention(meta, lay, out, range(bs))
    ref_k, ref_v = oracle.gather.kv_gather(
        u16(lay.k_stage)[None], u16(lay.v_stage)[None], u16(lay.k_pool)[None],
        u16(lay.v_pool)[None], meta.src_ids, meta.dst_ids)
    assert np.array_equal(u16(kp)[None], ref_k) and np.array_equal(u16(vp)[None], ref_v)


@pytest.mark.parametrize("hq,hkv,d", [(8, 2, 128), (16, 2, 128), (8, 1, 64), (4, 2, 64)])
@pytest.mark.parametrize("fused", [False, True])
def test_row_tiles(device, hq, hkv, d, fused):
    """Depths of one batch on both sides of every row-tile edge: each item takes the tiles its
    rows fill, whole and cut."""
    group = hq // hkv
    top = min(8, 64 // group - 1)
    depth = np.array([k for k in range(top + 1) for _ in range(2)])
    lens = np.where(np.arange(len(depth)) % 2, 40 + 37 * depth, 600 - 31 * depth)
    lens[-1] = 5000                                  # cut, beside whole ones
    for keep in (slice(0, -1), slice(None)):
        n, k = lens[keep], depth[keep]
        cfg = custom_config(seed=801, bs=len(n), num_q_heads=hq, num_kv_heads=hkv, head_dim=d,
                            vocab=0, n_arriving=0, pool_blocks=None, staging_order="shuffled")
        meta = make_meta(cfg, seq_lens=list(n), depth=k,
                         arriving=(np.arange(len(n)) % 3 != 1) & fused)
        lay = make_layer(cfg, meta, 0, device)
        args = (i32(meta.seq_lens, device), i32(meta.q_indptr, device), meta.max_q,
                meta.max_seq_len)
        table = i32(meta.block_table, device)
        if fused:
            out = nsd.gather_verify_attention(lay.q, lay.k_pool.clone(), lay.v_pool.clone(),
                                              lay.k_stage, lay.v_stage, table,
                                              i32(meta.stage_table, device), *args)
        else:
            out = nsd.verify_attention(lay.q, lay.k_pool, lay.v_pool, table, *args)
        torch.cuda.synchronize()
        check_attention(meta, lay, out, range(len(n)))


def test_more_items_than_a_grid_takes(device):
    """8192 requests of 2049 KV heads: a workgroup per item would be 2^32 threads, so the wave
    split takes them.  One token per context, so each output row is that token's V."""
    bs, hkv, d = 8192, 2049, 64
    gen = torch.Generator(device=device).manual_seed(5)
    k = torch.randn((2, hkv, d // 8, 16, 8), generator=gen, device=device).bfloat16()
    v = torch.randn((2, hkv, d, 16), generator=gen, device=device).bfloat16()
    q = torch.randn((bs, hkv, d), generator=gen, device=device).bfloat16()
    table = (torch.arange(bs, device=device, dtype=torch.int32) % 2)[:, None].contiguous()
    out = nsd.verify_attention(q, k, v, table,
                               torch.ones(bs, dtype=torch.int32, device=device),
                               torch.arange(bs + 1, dtype=torch.int32, device=device), 1, 1)
    torch.cuda.synchronize()
    for r in (0, 1):
        assert torch.equal(out[r::2], v[r, :, :, 0].expand(bs // 2, hkv, d))
