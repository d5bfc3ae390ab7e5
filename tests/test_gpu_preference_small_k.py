"""Dense preference score with a small top_k: the bound from the sampled keys lets through more candidates than 32 top_k, which
is no reason to evaluate the logits again in the exact form; short prompts, which take the exact form alone.  Oracle: float64."""
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
    """Lengths: 32 top_k and less, the last with every logit a candidate (944 at top_k = 1 to 1520 at 47), the first beyond."""
    print(f"case small k={top_k} n={n}", flush=True)
    rng = np.random.default_rng(100 * n + top_k)
    q = rng.standard_normal((16, 8, 128)).astype(np.float16)
    k = (rng.standard_normal((2, n, 128)) * 1.5).astype(np.float16)
    assert _exact_slabs(q, k, top_k)[0] == 0


@pytest.mark.parametrize("hq,hkv,n_q", [(2, 2, 16), (3, 1, 16), (8, 1, 16), (9, 1, 16), (17, 1, 16), (3, 3, 256)])
@pytest.mark.parametrize("n,top_k", [(2, 1), (16, 15), (17, 1), (129, 2), (129, 128), (700, 40), (1040, 300), (3071, 3070), (3072, 256),
                                     (3072, 1024), (3073, 1024)])
def test_short_prompts(hq, hkv, n_q, n, top_k):
    """Every number of rows per workgroup, chunks and their remainders, both sides of the length up to which the exact
    form is the only one, fewer block maxima than top_k and more."""
    print(f"case short {hq}/{hkv} n_q={n_q} n={n} k={top_k}", flush=True)
    rng = np.random.default_rng(n + hq)
    q = rng.standard_normal((n_q, hq, 128)).astype(np.float16)
    k = (rng.standard_normal((hkv, n, 128)) * 1.5).astype(np.float16)
    _exact_slabs(q, k, top_k)


@pytest.mark.parametrize("n,top_k", [(20000, 130), (20000, 180), (20000, 256), (20000, 400), (30000, 1024), (30000, 1200), (30000, 1700),
                                     (30000, 2000), (30000, 2400), (30000, 3000), (4096, 600), (4097, 600), (6144, 1500), (6145, 1500)])
def test_rows_of_every_final_kernel(n, top_k):
    """Numbers of candidates on both sides of what a final kernel keeps in registers (1024, 1536, 3072, 4096, 6144), all keys and most."""
    print(f"case final n={n} k={top_k}", flush=True)
    rng = np.random.default_rng(n + top_k)
    q = rng.standard_normal((16, 4, 128)).astype(np.float16)
    k = (rng.standard_normal((2, n, 128)) * 1.5).astype(np.float16)
    assert _exact_slabs(q, k, top_k)[0] == 0


def test_short_prompt_with_nan():
    rng = np.random.default_rng(2)
    q = rng.standard_normal((16, 4, 128)).astype(np.float16)
    k = rng.standard_normal((4, 400, 128)).astype(np.float16)
    want = preference.dense_preference(q, k, 64, SM)
    k[1, 77, 5] = np.nan      # a NaN logit in every row: no mass is reported outside
    dp = tkv.DensePreference(n_q_heads=4, n_kv_heads=4, n_q=16, top_k=64, capacity=400)
    for _ in range(2):
        got = dp.score(torch.from_numpy(q)[None].cuda(), torch.from_numpy(k.transpose(1, 0, 2).copy())[None].cuda(), SM)[0].cpu().numpy()
        assert got[1] == 0.0 and np.abs(got[[0, 2, 3]] - want[[0, 2, 3]]).max() <= 1e-4 * 16


def test_equal_logits_take_the_exact_form():
    """(The other way round, for the word that the test above reads: ties that no bound of the sample can divide.)"""
    rng = np.random.default_rng(1)
    q = rng.standard_normal((16, 8, 128)).astype(np.float16)
    k = np.repeat(rng.standard_normal((2, 1, 128)).astype(np.float16), 20000, axis=1)
    ran, slabs = _exact_slabs(q, k, 8)
    assert ran == slabs
