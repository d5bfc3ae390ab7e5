"""Sparse layers whose fetched rows are shared by several workgroups per head (few heads, many rows), and groups of 5 to 8
query heads in the one-launch step: both sides of each rule, lengths with fewer tokens than workgroups, ragged batches with
an empty sequence, queries, outputs and new rows at odd fp16 addresses.  Oracle: indices bit-exact, attention <= 2e-3."""
import numpy as np
import pytest
import torch

import paper_2505_19586_amd as tkv
from oracle import sparse
from synth import HeadShape, make_layer, static_channels

from gpu_util import attn_err, to_new, to_new_batch

pytestmark = pytest.mark.gpu
TOL = 2e-3
SM = 1.0 / np.sqrt(128.0)


def _odd(x):
    """The same values behind an address that is a multiple of 2 bytes only."""
    buf = torch.empty(x.numel() + 8, dtype=x.dtype, device=x.device)
    buf[1:1 + x.numel()] = x.view(-1)
    return buf[1:1 + x.numel()].view(x.shape)


def _check(layer, b, inp, ch, out, n):
    d = layer.desc
    torch.cuda.synchronize()
    if n == 0:
        assert (out[b] == 0).all() and int(layer.topk_count[b].sum()) == 0
        return
    k, v = inp.k[:, :n], inp.v[:, :n]
    idx, cnt = sparse.estimate_topk(inp.q, sparse.key_summary(k, ch), ch, n, top_k=d.top_k, n_sink=d.n_sink, n_window=d.n_window)
    assert np.array_equal(layer.topk_count[b].cpu().numpy(), cnt)
    assert np.array_equal(layer.topk_idx[b].cpu().numpy(), idx)
    want = sparse.sparse_attention(inp.q, k, v, idx, cnt, n, SM, n_sink=d.n_sink, n_window=d.n_window)
    assert attn_err(out[b], want) <= TOL


# n_sink + top_k + n_window: 256 is one workgroup per head, 257 five of them with fewer heads than query heads of a lane
@pytest.mark.parametrize("hq,hkv", [(8, 1), (4, 1), (16, 2), (21, 3), (28, 7), (64, 8), (5, 1)])
@pytest.mark.parametrize("top_k", [188, 189, 1024])
def test_rows_shared_by_workgroups(hq, hkv, top_k):
    shape = HeadShape(hq, hkv, 128)
    for n in (1, 69, 300, 3000):
        print(f"case split {hq}/{hkv} k={top_k} n={n}", flush=True)
        inp = make_layer(n + 1, shape=shape, seq=n % 31)
        ch = static_channels(inp.k, 12)
        layer = tkv.SparseLayer(n_q_heads=hq, n_kv_heads=hkv, n_channels=12, top_k=top_k, capacity=n + 8)
        layer.set_channels(ch[None])
        kd, vd = to_new(inp.k), to_new(inp.v)
        layer.append(kd[:, :n].contiguous(), vd[:, :n].contiguous())
        q = _odd(torch.from_numpy(inp.q)[None].cuda())
        for _ in range(2):  # (the counters are left clean)
            layer.estimate_topk(q)
            _check(layer, 0, inp, ch, layer.gather_attn(q, SM), n)
        out = _odd(torch.zeros_like(q))
        layer.decode(q, SM, _odd(kd[:, n:]), _odd(vd[:, n:]), out=out)
        _check(layer, 0, inp, ch, out, n + 1)
        layer.gather()
        _check(layer, 0, inp, ch, layer.attn(q, SM), n + 1)


@pytest.mark.parametrize("hq,hkv,batch", [(8, 1, 3), (8, 1, 9), (3, 1, 2)])
def test_ragged_batches(hq, hkv, batch):
    shape = HeadShape(hq, hkv, 128)
    lens = [0, 700, 68, 1500, 5, 900, 1, 1400, 333][:batch]
    print(f"case split ragged {hq}/{hkv} {lens}", flush=True)
    inps = [make_layer(max(n, 1), shape=shape, seq=b) for b, n in enumerate(lens)]
    chs = [static_channels(i.k, 8) for i in inps]
    layer = tkv.SparseLayer(n_q_heads=hq, n_kv_heads=hkv, n_channels=8, top_k=512, capacity=1512, batch=batch)
    layer.set_channels(np.stack(chs))
    layer.append(to_new_batch([i.k[:, :n] for i, n in zip(inps, lens)], max(lens)),
                 to_new_batch([i.v[:, :n] for i, n in zip(inps, lens)], max(lens)), n_valid=lens)
    q = torch.from_numpy(np.stack([i.q for i in inps])).cuda()
    out = layer.decode(q, SM)
    for b, inp in enumerate(inps):
        _check(layer, b, inp, chs[b], out, lens[b])
    out = layer.gather_attn(q, SM)
    for b, inp in enumerate(inps):
        _check(layer, b, inp, chs[b], out, lens[b])
