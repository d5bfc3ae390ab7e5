"""Sparse layers whose sequences fit one workgroup's share (up to 5120 tokens, 4096 with 5 to 8 query heads per KV head):
equal scores by the thousand, ragged batches on both sides of the limit, channel-major keys, the append by a workgroup
of its own and by the same one (many heads), no candidates.  Oracle: indices bit-exact, attention <= 2e-3."""
import numpy as np
import pytest
import torch

import paper_2505_19586_amd as tkv
from oracle import sparse
from synth import HeadShape, make_layer, static_channels

from gpu_util import attn_err, to_new_batch

pytestmark = pytest.mark.gpu
TOL = 2e-3
SM = 1.0 / np.sqrt(128.0)


@pytest.mark.parametrize("hq,hkv,ds", [(4, 1, 16), (8, 1, 12), (6, 2, 8)])
@pytest.mark.parametrize("lens", [(4096, 4095), (4097, 1), (5120, 4096, 0, 68, 69), (5121, 5120, 1024)])
def test_equal_scores_and_ragged_lengths(hq, hkv, ds, lens):
    """Coarse summaries: thousands of tokens share a score, or a score's leading bits."""
    batch, cap = len(lens), 5128
    rng = np.random.default_rng(sum(lens) + hq)
    q = rng.standard_normal((batch, hq, 128)).astype(np.float16)
    ch = np.sort(np.stack([[rng.permutation(128)[:ds] for _ in range(hkv)] for _ in range(batch)]), axis=2).astype(np.int32)
    coarse = rng.integers(0, 2, (batch, hkv, cap, 1)) * np.ones(ds)  # two scores
    fine = 1.0 + rng.integers(0, 3000, (batch, hkv, cap, 1)) * np.eye(ds)[0] * 2.0 ** -10  # near each other
    for name, summary in (("two", coarse), ("near", fine), ("zero", 0.0 * fine)):
        summary = summary.astype(np.float16)
        for top_k in (1, 1500, 4096):
            print(f"case one share {hq}/{hkv} ds={ds} lens={lens} {name} k={top_k}", flush=True)
            layer = tkv.SparseLayer(n_q_heads=hq, n_kv_heads=hkv, n_channels=ds, top_k=top_k, capacity=cap, batch=batch)
            layer.set_channels(ch)
            layer.key_summary.copy_(torch.from_numpy(summary))
            layer.seq_len[:] = lens
            for _ in range(2):  # (the counters are left clean)
                layer.topk_idx.fill_(-7)
                idx, cnt = layer.estimate_topk(torch.from_numpy(q).cuda())
                torch.cuda.synchronize()
                for b, n in enumerate(lens):
                    want_idx, want_cnt = sparse.estimate_topk(q[b], summary[b], ch[b], n, top_k=top_k, n_sink=4, n_window=64)
                    assert np.array_equal(cnt[b].cpu().numpy(), want_cnt)
                    assert np.array_equal(idx[b].cpu().numpy(), want_idx)


# up to 128 (sequence, KV head) pairs leave a compute unit for each one's append, 129 and 130 do not
@pytest.mark.parametrize("hq,hkv,batch", [(8, 2, 3), (6, 1, 64), (65, 65, 2), (15, 3, 43)])
def test_decode_appends_in_the_same_launch(hq, hkv, batch):
    shape = HeadShape(hq, hkv, 128)
    lens = [(0, 700, 68, 1, 90, 200)[b % 6] for b in range(batch)]
    print(f"case one share decode {hq}/{hkv} batch={batch}", flush=True)
    inps = [make_layer(702, shape=shape, seq=b % 6) for b in range(min(batch, 6))]
    chs = [static_channels(i.k, 8) for i in inps]
    layer = tkv.SparseLayer(n_q_heads=hq, n_kv_heads=hkv, n_channels=8, top_k=64, capacity=704, batch=batch)
    layer.set_channels(np.stack([chs[b % 6] for b in range(batch)]))
    cut = lambda x, b, a, e: x[:, a:e]
    rows = lambda what, a, e: [cut(getattr(inps[b % 6], what), b, *((0, lens[b]) if a is None else (lens[b] + a, lens[b] + e)))
                               for b in range(batch)]
    layer.append(to_new_batch(rows("k", None, None), 700), to_new_batch(rows("v", None, None), 700), n_valid=lens)
    q = torch.from_numpy(np.stack([inps[b % 6].q for b in range(batch)])).cuda()
    for step in range(2):
        out = layer.decode(q, SM, to_new_batch(rows("k", step, step + 1), 1), to_new_batch(rows("v", step, step + 1), 1))
        torch.cuda.synchronize()
        for b in range(batch):
            inp, ch, n = inps[b % 6], chs[b % 6], lens[b] + step + 1
            k, v = inp.k[:, :n], inp.v[:, :n]
            idx, cnt = sparse.estimate_topk(inp.q, sparse.key_summary(k, ch), ch, n, top_k=64, n_sink=4, n_window=64)
            assert np.array_equal(layer.topk_count[b].cpu().numpy(), cnt)
            assert np.array_equal(layer.topk_idx[b].cpu().numpy(), idx)
            want = sparse.sparse_attention(inp.q, k, v, idx, cnt, n, SM, n_sink=4, n_window=64)
            assert attn_err(out[b], want) <= TOL
