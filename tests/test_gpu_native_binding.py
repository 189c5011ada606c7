"""The native marshalling against the Python one: a tensor subclass is not taken
natively, so the same calls with one go through ctypes; outputs are identical,
with and without the caller's buffers, and a wrong argument raises the same."""
import ctypes
import gc

import numpy as np
import pytest
import torch

import paper_2609_29364_amd as nsd
from paper_2609_29364_amd.round import draft_stage, fused_tables, verify_round
from workload import custom_config, make_accept, make_draft, make_layer, make_meta
from parity import i32

pytestmark = pytest.mark.gpu


class Plain(torch.Tensor):
    """A subclass without behaviour of its own."""


def both(call, *tensors):
    """call(*tensors) natively and, with the first tensor a subclass, through ctypes."""
    a = call(*[t.clone() for t in tensors])
    other = [t.clone() for t in tensors]
    other[0] = other[0].as_subclass(Plain)
    b = call(*other)
    torch.cuda.synchronize()
    flat = lambda v: [x.as_subclass(torch.Tensor) for x in v if x is not None]
    for x, y in zip(flat(a), flat(b), strict=True):
        assert torch.equal(x.view(torch.int16 if x.dtype == torch.bfloat16 else x.dtype),
                           y.view(torch.int16 if y.dtype == torch.bfloat16 else y.dtype))


def setup(device, bs=9, layers=2, vocab=1000, n_arriving=4):
    cfg = custom_config(seed=31, bs=bs, num_layers=layers, num_q_heads=8, num_kv_heads=2,
                        head_dim=128, vocab=vocab, n_arriving=n_arriving, pool_blocks=None,
                        ctx_lo=20, ctx_hi=300, k_lo=0, k_hi=5)
    meta = make_meta(cfg)
    lay = [make_layer(cfg, meta, l, device) for l in range(layers)]
    stack = lambda n: torch.nan_to_num(torch.stack([getattr(l, n) for l in lay])).contiguous()
    return cfg, meta, [stack(n) for n in ("k_pool", "v_pool", "k_stage", "v_stage", "q")]


@pytest.mark.parametrize("buffers", [False, True])
def test_calls(device, buffers):
    cfg, meta, (k, v, ks, vs, q) = setup(device)
    table, stage = i32(meta.block_table, device), i32(meta.stage_table, device)
    lens, qi = i32(meta.seq_lens, device), i32(meta.q_indptr, device)
    src, dst = i32(meta.src_ids, device), i32(meta.dst_ids, device)
    more = (lambda t: dict(out=torch.empty_like(t), workspace=nsd.new_workspace(
        nsd.verify_attention_workspace_size(cfg.bs, 8, 2, 128, meta.max_q, meta.max_seq_len),
        device))) if buffers else (lambda t: {})
    both(lambda q, k, v: [nsd.verify_attention(q, k, v, table, lens, qi, meta.max_q,
                                               meta.max_seq_len, **more(q[:]))], q[0], k[0], v[0])
    both(lambda q, k, v: [nsd.gather_verify_attention(
        q, k, v, ks[0], vs[0], table, stage, lens, qi, meta.max_q, meta.max_seq_len,
        **more(q[:])), k, v], q[0], k[0], v[0])
    both(lambda k, v: [*nsd.kv_gather(ks, vs, k, v, src, dst)], k, v)
    both(lambda k, v: [*nsd.kv_gather(ks, vs, k, v, src, dst, layer0=1, n_layers=1)], k, v)
    both(lambda k, v: [*nsd.kv_gather(ks[0], vs[0], k, v, src, dst)], k[0], v[0])
    rows = torch.randn(meta.total_q, 2, 128, device=device).bfloat16()
    both(lambda k, v: [nsd.kv_append(k, v, rows, rows, table, lens, qi), k, v], k[0], v[0])
    a = make_accept(cfg, meta, device)
    both(lambda p: [*nsd.spec_accept(p, a.q_draft, a.draft_tokens, a.uniforms, qi,
                                     meta.max_q - 1)], a.p_target)
    acc = torch.zeros(cfg.bs, dtype=torch.int32, device=device)
    both(lambda l: [nsd.commit_lengths(l, qi, acc)], lens)
    p3 = a.p_target[:8].view(2, 4, -1)
    both(lambda p: [nsd.sample(p.view(2, 4, -1)[:, 1], a.uniforms[:2])], p3.contiguous())


@pytest.mark.parametrize("bs", [9, 17])
@pytest.mark.parametrize("window", [False, True])
@pytest.mark.parametrize("prepare", ["auto", "fused", "gather"])
def test_round(device, bs, window, prepare):
    cfg, meta, (k, v, ks, vs, q) = setup(device, bs=bs)
    table, stage = i32(meta.block_table, device), i32(meta.stage_table, device)
    ws = nsd.new_workspace(nsd.verify_attention_workspace_size(
        bs, 8, 2, 128, meta.max_q, meta.max_seq_len), device)
    a = make_accept(cfg, meta, device)
    kv = [tuple(torch.randn(meta.total_q, 2, 128, device=device).bfloat16() for _ in range(2))
          for _ in range(2)] if window else None

    def call(k, v, ks, vs):
        committed = torch.zeros(bs, dtype=torch.int32, device=device)
        r = verify_round(k, v, ks, vs, i32(meta.src_ids, device), i32(meta.dst_ids, device), q,
                         table, i32(meta.seq_lens, device), i32(meta.q_indptr, device),
                         meta.max_q, meta.max_seq_len, out=torch.zeros_like(q), workspace=ws,
                         accept=(a.p_target, a.q_draft, a.draft_tokens, a.uniforms,
                                 meta.max_q - 1),
                         stage_table=stage, window_kv=kv, committed=committed, prepare=prepare)
        return [*r, committed, k, v, ks, vs]

    both(call, k, v, ks, vs)


@pytest.mark.parametrize("n_arriving", [0, 3])
def test_draft(device, n_arriving):
    cfg = custom_config(seed=33, bs=7, num_q_heads=4, num_kv_heads=2, head_dim=64, vocab=0,
                        n_arriving=n_arriving, pool_blocks=None, ctx_lo=20, ctx_hi=300, k_lo=0,
                        k_hi=0)
    dd = make_draft(cfg, 3, 1000, device)
    m, lay = dd.meta, dd.layer
    ws = nsd.new_workspace(nsd.verify_attention_workspace_size(7, 4, 2, 64, 1, m.max_seq_len),
                           device)

    def call(k, v):
        r = draft_stage(k, v, dd.q, dd.k_new, dd.v_new, dd.probs, dd.uniforms,
                        i32(m.block_table, device), dd.lens, i32(m.q_indptr, device),
                        m.max_seq_len, k_stage=lay.k_stage.clone(), v_stage=lay.v_stage.clone(),
                        stage_table=i32(m.stage_table, device), workspace=ws)
        return [*r, torch.nan_to_num(k), torch.nan_to_num(v)]

    both(call, lay.k_pool, lay.v_pool)


def test_draft_small_sample_workspace(device):
    """A sample workspace too small for one step is refused, whatever the others hold; one for
    a single step is enough."""
    cfg = custom_config(seed=34, bs=3, num_q_heads=4, num_kv_heads=2, head_dim=64, vocab=0,
                        n_arriving=0, pool_blocks=None, ctx_lo=20, ctx_hi=300, k_lo=0, k_hi=0)
    dd = make_draft(cfg, 3, 40000, device)
    m, lay = dd.meta, dd.layer
    ws = nsd.new_workspace(nsd.verify_attention_workspace_size(3, 4, 2, 64, 1, m.max_seq_len),
                           device)
    need = nsd.accept_workspace_size(3, 40000)

    def call(size):
        return draft_stage(lay.k_pool, lay.v_pool, dd.q, dd.k_new, dd.v_new, dd.probs,
                           dd.uniforms, i32(m.block_table, device), dd.lens,
                           i32(m.q_indptr, device), m.max_seq_len, workspace=ws,
                           sample_workspace=torch.empty(size, dtype=torch.uint8,
                                                        device=device))[1]

    with pytest.raises(nsd.NsdError) as e:
        call(need - 1)
    assert e.value.status == 4
    assert torch.equal(call(need), call(4 * need))


@pytest.mark.parametrize("layer0", [-1, -2**31, 3, 2**31 - 1])
def test_gather_layer_range(device, layer0):
    cfg, meta, (k, v, ks, vs, q) = setup(device)
    src, dst = i32(meta.src_ids, device), i32(meta.dst_ids, device)
    before = k.clone()
    with pytest.raises(nsd.NsdError):
        nsd.kv_gather(ks, vs, k, v, src, dst, layer0=layer0)
    torch.cuda.synchronize()
    assert torch.equal(k, before)


def test_faults_raise_the_same(device):
    cfg, meta, (k, v, ks, vs, q) = setup(device)
    table, lens, qi = (i32(x, device) for x in (meta.block_table, meta.seq_lens, meta.q_indptr))
    good = [q[0], k[0], v[0], table, lens, qi, meta.max_q, meta.max_seq_len]
    for at, bad, error in [(0, q[0].float(), TypeError), (0, q[0].cpu(), ValueError),
                           (1, k[0].transpose(0, 1), ValueError), (3, table[:-1], ValueError),
                           (4, lens.long(), TypeError), (6, 1000, nsd.NsdError)]:
        args = list(good)
        args[at] = bad
        with pytest.raises(error):
            nsd.verify_attention(*args)
    with pytest.raises(nsd.NsdError) as e:
        nsd.verify_attention(*good, workspace=torch.empty(16, dtype=torch.uint8, device=device))
    assert e.value.status == 4 and "workspace" in str(e.value)


def test_a_list_changed_during_the_call(device):
    """The native round runs without the interpreter lock; rows taken out of the caller's list
    meanwhile stay alive until it has submitted its last launch."""
    cfg, meta, (k, v, ks, vs, q) = setup(device)
    ws = nsd.new_workspace(nsd.verify_attention_workspace_size(
        cfg.bs, 8, 2, 128, meta.max_q, meta.max_seq_len), device)
    row = lambda: torch.zeros((meta.total_q, 2, 128), dtype=torch.bfloat16, device=device)
    rows = [[row(), row()] for _ in range(2)]
    seen = []
    res, args = nsd._SIGS["nsd_kv_append_layers"]

    def append(*a):      # in the entry point's place: another thread empties the list
        before = torch.cuda.memory_allocated()
        rows.clear()
        seen.append(torch.cuda.memory_allocated() - before)
        return 0

    callback = ctypes.CFUNCTYPE(res, *args)(append)
    at = lambda f: ctypes.cast(f, ctypes.c_void_p).value
    real = [at(getattr(nsd.lib(), f)) for f in nsd._BOUND]
    native = nsd._native()
    gc.collect()         # tensors of other tests' cycles go now, not inside the callback
    gc.disable()
    try:
        native.bind(tuple(at(callback) if f == "nsd_kv_append_layers" else r
                          for f, r in zip(nsd._BOUND, real)))
        verify_round(k, v, ks, vs, i32(meta.src_ids, device), i32(meta.dst_ids, device), q,
                     i32(meta.block_table, device), i32(meta.seq_lens, device),
                     i32(meta.q_indptr, device), meta.max_q, meta.max_seq_len,
                     out=torch.zeros_like(q), workspace=ws, window_kv=rows)
    finally:
        gc.enable()
        native.bind(tuple(real))
    torch.cuda.synchronize()
    assert seen == [0] and not rows
