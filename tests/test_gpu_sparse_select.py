"""Selection of sparse layers at the sizes where its paths change: few tokens per share, k up to all candidates, lists that
fill their part of the last workgroup's round.  Scores of random summaries against the oracle, indices bit-exact."""
import numpy as np
import pytest
import torch

import paper_2505_19586_amd as tkv
from oracle import sparse

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,ds", [(32, 8, 16), (8, 1, 12), (6, 2, 8)])
@pytest.mark.parametrize("n", [69, 1023, 1025, 2000, 4097, 5120, 5121, 6000, 12000, 40000])
def test_counts_of_selected_tokens(hq, hkv, ds, n):
    rng = np.random.default_rng(n + hq)
    summary = rng.standard_normal((hkv, n, ds)).astype(np.float16)
    q = rng.standard_normal((hq, 128)).astype(np.float16)
    ch = np.sort(np.stack([rng.permutation(128)[:ds] for _ in range(hkv)]), axis=1).astype(np.int32)
    qd = torch.from_numpy(q)[None].cuda()
    kv = torch.zeros(hkv * (n + 16) * 256, dtype=torch.float16, pin_memory=True)
    for top_k in (1, 16, 64, 128, 512, 1024, 2048, 4096):
        print(f"case select {hq}/{hkv} ds={ds} n={n} k={top_k}", flush=True)
        layer = tkv.SparseLayer(n_q_heads=hq, n_kv_heads=hkv, n_channels=ds, top_k=top_k, capacity=n, kv_host=kv[:hkv * n * 256])
        layer.set_channels(ch[None])
        layer.key_summary[0].copy_(torch.from_numpy(summary))
        layer.seq_len[:] = n
        want_idx, want_cnt = sparse.estimate_topk(q, summary, ch, n, top_k=top_k, n_sink=4, n_window=64)
        for _ in range(2):  # (the counters are left clean)
            layer.topk_idx.fill_(-7)
            idx, cnt = layer.estimate_topk(qd)
            torch.cuda.synchronize()
            assert np.array_equal(cnt[0].cpu().numpy(), want_cnt)
            assert np.array_equal(idx[0].cpu().numpy(), want_idx)
