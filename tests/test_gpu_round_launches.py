"""The launches a round and a draft stage share over layers and steps, each
against the calls they stand for: the append of all layers into two banks, the
acceptance that commits lengths, the draws of all steps."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2609_29364_amd as nsd
from parity import i32, u16

pytestmark = pytest.mark.gpu


def _bits(rng, *shape):
    return torch.from_numpy(rng.integers(-30000, 30000, size=shape,
                                         dtype=np.int16)).view(torch.bfloat16)


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("layers,shift", [(1, 0), (2, 1), (33, 0)])   # 32 layers a launch
def test_append_layers(device, head_dim, layers, shift):
    """Requests 0 and 2 in the pool, 1 and 3 in the staging bank; windows inside a block, over
    a boundary and over three blocks; rows at any 2-byte alignment."""
    rng = np.random.default_rng(layers)
    hkv, nb, ns = 3, 9, 7
    lens, nqs = [19, 16, 48, 33], [5, 1, 40, 6]
    pool_t = np.array([[3, 4, -1], [-1] * 3, [5, 6, 7], [-1] * 3], dtype=np.int32)
    stage_t = np.array([[-1] * 3, [1, -1, -1], [-1, ns, -1], [2, 3, 4]], dtype=np.int32)
    qi = np.concatenate([[0], np.cumsum(nqs)]).astype(np.int32)
    planes = lambda n: (_bits(rng, layers, n, hkv, head_dim // 8, 16, 8),
                        _bits(rng, layers, n, hkv, head_dim, 16))
    banks = [planes(nb), planes(ns)]
    new = [[_bits(rng, int(qi[-1]), hkv, head_dim) for _ in range(2)] for _ in range(layers)]

    def place(t):      # on the device, `shift` elements past an aligned address
        flat = torch.empty(t.numel() + shift, dtype=t.dtype, device=device)
        flat[shift:] = t.flatten()
        return flat[shift:]

    rows = [[place(t) for t in kv] for kv in new]
    k, v, ks, vs = (t.to(device) for pair in banks for t in pair)
    ptrs = [(ctypes.c_void_p * layers)(*[kv[i].data_ptr() for kv in rows]) for i in range(2)]
    tables = [i32(t, device) for t in (pool_t, stage_t)]
    meta = [i32(np.array(lens), device), i32(qi, device)]
    st = nsd.lib().nsd_kv_append_layers(
        k.data_ptr(), v.data_ptr(), nb, tables[0].data_ptr(), ks.data_ptr(), vs.data_ptr(), ns,
        tables[1].data_ptr(), layers, ptrs[0], ptrs[1], 3, meta[0].data_ptr(),
        meta[1].data_ptr(), 4, int(qi[-1]), hkv, 16, head_dim,
        torch.cuda.current_stream().cuda_stream)
    assert st == 0
    torch.cuda.synchronize()
    for bank, table, out in ((banks[0], pool_t, (k, v)), (banks[1], stage_t, (ks, vs))):
        # the oracle takes ids in range: the others write to a spare block it appends
        n = bank[0].shape[1]
        ids = np.where((table >= 0) & (table < n), table, n)
        for l in range(layers):
            spare = [np.concatenate([u16(t[l]), np.zeros_like(u16(t[l][:1]))]) for t in bank]
            ref = oracle.commit.kv_append(*spare, u16(new[l][0]), u16(new[l][1]), ids, lens, qi)
            for got, want in zip(out, ref):
                assert np.array_equal(u16(got[l]), want[:n])


@pytest.mark.parametrize("bs,vocab", [(5, 1000), (5, 40000), (300, 20000), (256, 20000)])
def test_accept_commit(device, bs, vocab):
    """One workgroup a row and rows spread over several: the lengths the two calls give, in
    place too."""
    g = torch.Generator(device=device).manual_seed(bs)
    depth = np.arange(bs) % 6
    indptr = i32(np.concatenate([[0], np.cumsum(depth + 1)]), device)
    total = int(indptr[-1])
    p = torch.rand((total, vocab), generator=g, device=device)
    q = torch.rand((total - bs, vocab), generator=g, device=device)
    x = torch.randint(0, vocab, (total - bs,), generator=g, device=device, dtype=torch.int32)
    u = torch.rand(total, generator=g, device=device)
    lens = torch.randint(100, 1000, (bs,), generator=g, device=device, dtype=torch.int32)
    acc, tok = nsd.spec_accept(p, q, x, u, indptr, 5)
    want = nsd.commit_lengths(lens, indptr, acc)
    ws = torch.empty(nsd.accept_workspace_size(bs, vocab), dtype=torch.uint8, device=device)
    for new in (torch.zeros_like(lens), lens):
        acc2, tok2 = torch.full_like(acc, -7), torch.full_like(tok, -7)
        st = nsd.lib().nsd_spec_accept_commit(
            p.data_ptr(), q.data_ptr(), x.data_ptr(), u.data_ptr(), indptr.data_ptr(), bs, vocab,
            5, acc2.data_ptr(), tok2.data_ptr(), lens.data_ptr(), new.data_ptr(), ws.data_ptr(),
            ws.numel(), torch.cuda.current_stream().cuda_stream)
        assert st == 0
        torch.cuda.synchronize()
        assert torch.equal(acc, acc2) and torch.equal(tok, tok2) and torch.equal(new, want)


@pytest.mark.parametrize("n,steps,vocab", [(1, 1, 4), (3, 5, 1000), (7, 3, 40000),
                                           (64, 4, 20000), (90, 4, 20000)])
def test_sample_steps(device, n, steps, vocab):
    """Rows and tokens inside wider buffers; both ways a batch is laid over the CUs."""
    g = torch.Generator(device=device).manual_seed(n)
    p = torch.rand((n, steps + 1, vocab), generator=g, device=device)
    u = torch.rand((steps, n), generator=g, device=device)
    want = torch.full((n, steps + 1), -7, dtype=torch.int32, device=device)
    got = want.clone()
    for i in range(steps):
        nsd.sample(p[:, i], u[i], out=want[:, i])
    ws = torch.empty(nsd.accept_workspace_size(n * steps, vocab), dtype=torch.uint8,
                     device=device)
    st = nsd.lib().nsd_sample_steps(p.data_ptr(), p.stride(0), u.data_ptr(), n, steps, vocab,
                                    got.data_ptr(), steps + 1, ws.data_ptr(), ws.numel(),
                                    torch.cuda.current_stream().cuda_stream)
    assert st == 0
    torch.cuda.synchronize()
    assert torch.equal(got, want)
