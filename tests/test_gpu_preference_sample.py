"""Dense preference score where the bound from the sampled keys matters: every number of query rows per KV head, prompts
at the edges of chunks, strata and the all-candidates rule; prompts made against the sample (its bound fails, the exact
form takes over), outliers it cannot see, candidates crowded in one workgroup, NaN and infinite keys.  Oracle: float64."""
import numpy as np
import pytest
import torch

import paper_2505_19586_amd as tkv
from oracle import preference

pytestmark = pytest.mark.gpu
SM = 1.0 / np.sqrt(128.0)


def sampled_keys(n):
    """The kernels' sample: one key of every 16."""
    x = np.arange((n + 15) // 16, dtype=np.uint64)
    m = np.uint64(0xFFFFFFFF)
    i = x.copy()
    x = (x * np.uint64(0x9E3779B9) + np.uint64(0x3C6EF372)) & m
    x = ((x ^ (x >> np.uint64(16))) * np.uint64(0xBB67AE85)) & m
    x = ((x ^ (x >> np.uint64(16))) * np.uint64(0x6A09E667)) & m
    s = 16 * i + (x >> np.uint64(28))
    return s[s < n].astype(np.int64)


def _score(q_last, k, top_k, capacity=None):
    """q_last [n_q, Hq, D], k [Hkv, n, D]; two calls, bit for bit the same."""
    n_q, hq, _ = q_last.shape
    hkv, n, _ = k.shape
    dp = tkv.DensePreference(n_q_heads=hq, n_kv_heads=hkv, n_q=n_q, top_k=top_k, capacity=capacity or n)
    qd = torch.from_numpy(q_last)[None].contiguous().cuda()
    kd = torch.from_numpy(np.ascontiguousarray(k.transpose(1, 0, 2)))[None].contiguous().cuda()
    out, out2 = dp.score(qd, kd, SM), dp.score(qd, kd, SM)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int32), out2.view(torch.int32))
    return out[0].cpu().numpy().astype(np.float64)


def _check(q_last, k, top_k, capacity=None):
    got, want = _score(q_last, k, top_k, capacity), preference.dense_preference(q_last, k, top_k, SM)
    assert np.abs(got - want).max() <= 1e-4 * q_last.shape[0]


@pytest.mark.parametrize("hq,hkv,n_q", [(2, 2, 16), (4, 4, 32), (6, 2, 16), (8, 2, 16), (6, 1, 16), (8, 1, 16), (9, 1, 16),
                                        (16, 1, 16), (17, 1, 16), (3, 3, 256)])
@pytest.mark.parametrize("n,top_k", [(127, 16), (129, 128), (2047, 64), (2049, 2048), (5000, 300), (9001, 512)])
def test_rows_and_lengths(hq, hkv, n_q, n, top_k):
    print(f"case sample {hq}/{hkv} n_q={n_q} n={n} k={top_k}", flush=True)
    rng = np.random.default_rng(n + hq)
    q = rng.standard_normal((n_q, hq, 128)).astype(np.float16)
    k = (rng.standard_normal((hkv, n, 128)) * 1.5).astype(np.float16)
    _check(q, k, top_k, capacity=n + 77)


def _along(rng, levels, hq=8, hkv=2, n_q=16):
    """Keys whose logits are about levels[token] for every query row."""
    u = rng.standard_normal((hkv, 1, 128))
    u /= np.linalg.norm(u, axis=-1, keepdims=True)
    noise = 0.02 * rng.standard_normal((hkv, len(levels), 128))
    k = (np.asarray(levels)[None, :, None] * u + noise).astype(np.float16)
    q = (np.sqrt(128.0) * np.repeat(u[:, 0], hq // hkv, axis=0)[None] + 0.02 * rng.standard_normal((n_q, hq, 128))).astype(np.float16)
    return q, k


@pytest.mark.parametrize("n,top_k", [(20000, 512), (70000, 256)])
def test_prompts_made_against_the_sample(n, top_k):
    rng = np.random.default_rng(n)
    s = sampled_keys(n)
    base = rng.standard_normal(n)
    high = base.copy()
    high[s] += 6.0            # only sampled keys are large: too few candidates above their bound
    _check(*_along(rng, high), top_k)
    low = base + 4.0
    low[s] = -4.0             # the sample sees none of the large ones: more candidates than there is room for
    _check(*_along(rng, low), top_k)


@pytest.mark.parametrize("jump", [3.0, 30.0, 70.0, 140.0, 400.0])
def test_outliers_that_the_sample_misses(jump):
    """The row maximum lies `jump` (units of the logit) above the sampled one: denominators against the sample's reference,
    beyond float's range from about 88 on."""
    n = 9000
    rng = np.random.default_rng(int(jump))
    levels = rng.standard_normal(n)
    free = np.setdiff1d(np.arange(n), sampled_keys(n))
    levels[free[[3, 4000, 8000]]] = [jump, jump - 0.5, jump - 1.0]
    _check(*_along(rng, levels), 128)
    _check(*_along(rng, levels), 2)


def test_candidates_crowded_in_one_workgroup():
    """2 KV heads: chunks r, r + P, ... of 128 keys belong to workgroup r; all large keys lie in those of one."""
    n = 64 * 1024
    rng = np.random.default_rng(5)
    levels = rng.standard_normal(n)
    chunk = np.arange(n) // 128
    for P in (64, 128):
        crowded = levels + 5.0 * (chunk % P == 3)
        _check(*_along(rng, crowded), 500)


def test_nan_and_infinite_keys():
    n = 4000
    rng = np.random.default_rng(3)
    q = rng.standard_normal((16, 4, 128)).astype(np.float16)
    k = rng.standard_normal((4, n, 128)).astype(np.float16)
    want = preference.dense_preference(q, k, 64, SM)
    k[1, 77, 5] = np.nan      # a NaN logit in every row: no mass is reported outside
    k[2, 1234, 9] = np.inf    # +inf in the rows of positive q (their maximum: the same), -inf in the others (no weight)
    finite = q[:, 2:3][q[:, 2, 9] < 0]
    others = np.delete(k[2:3], 1234, axis=1)
    want_2 = preference.dense_preference(finite, others, 64, SM)[0]
    got = _score(q, k, 64)
    assert np.abs(got[[0, 3]] - want[[0, 3]]).max() <= 1e-4 * 16
    assert got[1] == 0.0 and abs(got[2] - want_2) <= 1e-4 * 16
