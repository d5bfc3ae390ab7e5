"""Dense preference score with a small top_k: the bound from the sampled keys lets through more candidates than 32 top_k (where
the prompt is short, every logit), which is no reason to evaluate the logits again in the exact form.  Oracle: float64."""
import numpy as np
import pytest
import torch

import paper_2505_19586_amd as tkv
from oracle import preference

pytestmark = pytest.mark.gpu
SM = 1.0 / np.sqrt(128.0)


def _exact_slabs(q_last, k, top_k):
    """Score checked against the oracle; slabs of rows that took the exact form."""
    (n_q, hq, _), (hkv, n, _) = q_last.shape, k.shape
    dp = tkv.DensePreference(n_q_heads=hq, n_kv_heads=hkv, n_q=n_q, top_k=top_k, capacity=n)
    qd = torch.from_numpy(q_last)[None].contiguous().cuda()
    kd = torch.from_numpy(np.ascontiguousarray(k.transpose(1, 0, 2)))[None].contiguous().cuda()
    got = dp.score(qd, kd, SM)[0].cpu().numpy().astype(np.float64)
    assert np.abs(got - preference.dense_preference(q_last, k, top_k, SM)).max() <= 1e-4 * n_q
    # the workspace begins with four words per row (the candidates' counters), then one per slab of up to 256 rows: did
    # the exact form run for it
    rows = hq // hkv * n_q
    slabs = hkv * ((rows + 255) // 256)
    words = dp.workspace[16 * hkv * rows:][:4 * slabs].view(torch.int32)
    return int(words.ne(0).sum()), slabs


@pytest.mark.parametrize("top_k", [1, 2, 5, 8, 9, 16, 17, 32, 47, 48])
@pytest.mark.parametrize("n", [33, 300, 944, 945, 1136, 1392, 1520, 1521, 6000, 20000])
def test_plain_prompts_need_one_evaluation(top_k, n):
    """Lengths: 32 top_k and less, the last of the all-candidates rule (944 at top_k = 1 to 1520 at 47), the first beyond."""
    print(f"case small k={top_k} n={n}", flush=True)
    rng = np.random.default_rng(100 * n + top_k)
    q = rng.standard_normal((16, 8, 128)).astype(np.float16)
    k = (rng.standard_normal((2, n, 128)) * 1.5).astype(np.float16)
    assert _exact_slabs(q, k, top_k)[0] == 0


def test_equal_logits_take_the_exact_form():
    """(The other way round, for the word that the test above reads: ties that no bound of the sample can divide.)"""
    rng = np.random.default_rng(1)
    q = rng.standard_normal((16, 8, 128)).astype(np.float16)
    k = np.repeat(rng.standard_normal((2, 1, 128)).astype(np.float16), 20000, axis=1)
    ran, slabs = _exact_slabs(q, k, 8)
    assert ran == slabs
