"""tkv_quant_decode in the steps that complete a quantization group: the attention launch quantizes it.  The cache must be what
the append alone makes of it, bit for bit, and the output the attention's over that cache."""
import numpy as np
import pytest
import torch

import paper_2505_19586_amd as tkv
from gpu_util import attn_err

pytestmark = pytest.mark.gpu
SM = 1.0 / np.sqrt(128.0)


def _rows(rng, batch, n, hkv, special):
    x = rng.standard_normal((batch, n, hkv, 128)).astype(np.float16)
    x[:, :, :, 3] *= 10
    if special:  # zeros of both signs, constant channels and tokens, subnormal ranges
        x[:, :, :, 5] = np.where(rng.random((batch, n, hkv)) < 0.5, np.float16(0.0), np.float16(-0.0))
        x[:, :, :, 7] = np.float16(1.5)
        x[:, n // 2] = np.float16(-2.0)
        x[:, :, :, 9] = (rng.integers(0, 5, (batch, n, hkv)) * 6e-8).astype(np.float16)
    return torch.from_numpy(x).cuda()


def _pair(hq, hkv, bits, group, residual, batch, lens, add, special=False, capacity=None):
    rng = np.random.default_rng(hq * 131 + group + lens[0])
    top = max(lens)
    k, v = _rows(rng, batch, top, hkv, special), _rows(rng, batch, top, hkv, special)
    kn, vn = _rows(rng, batch, add, hkv, False), _rows(rng, batch, add, hkv, False)
    q = torch.from_numpy(rng.standard_normal((batch, hq, 128)).astype(np.float16)).cuda()
    made = []
    for _ in range(2):
        L = tkv.QuantLayer(n_q_heads=hq, n_kv_heads=hkv, bits=bits, group_size=group, residual=residual,
                           capacity=capacity or (top + add + 2 * group) // group * group, batch=batch)
        L.append(k, v, n_valid=np.array(lens, dtype=np.int32))
        made.append(L)
    return made, q, kn, vn


def _same(a, b):
    for name in a.buffers:
        x, y = a.buffers[name].view(torch.uint8), b.buffers[name].view(torch.uint8)
        assert torch.equal(x, y), name


def _check(hq, hkv, bits, group, residual, lens, add, special=False):
    print(f"case complete {hq}/{hkv} {bits}/{group} w={residual} lens={lens} add={add}", flush=True)
    (one, two), q, kn, vn = _pair(hq, hkv, bits, group, residual, len(lens), lens, add, special)
    out = one.decode(q, SM, kn, vn)
    two.append(kn, vn)
    ref = two.attn_decode(q, SM)
    torch.cuda.synchronize()
    assert list(one.seq_len) == [n + add for n in lens] == list(two.seq_len)
    _same(one, two)
    assert torch.isfinite(out).all()
    for b in range(len(lens)):
        assert attn_err(out[b], ref[b].float().cpu().numpy().astype(np.float64)) <= 2e-3
    again = one.attn_decode(q, SM)   # the cache as the next call finds it; the counters were left clean
    torch.cuda.synchronize()
    for b in range(len(lens)):
        assert attn_err(again[b], ref[b].float().cpu().numpy().astype(np.float64)) <= 2e-3


SETTINGS = [(2, 32), (4, 32), (1, 64), (2, 64)]


@pytest.mark.parametrize("bits,group", SETTINGS)
@pytest.mark.parametrize("hq,hkv", [(8, 2), (8, 1), (3, 3), (12, 2)])
def test_one_token(bits, group, hq, hkv):
    for residual in (group, 128, 256):
        for m in (1, 2, 5, 30, 200):  # completes group m - 1: the first one, one chunk, several chunks
            _check(hq, hkv, bits, group, residual, [residual + group * m - 1], 1, special=m == 5)


@pytest.mark.parametrize("bits,group", SETTINGS)
@pytest.mark.parametrize("add", [2, 3, 33, 64, 129])
def test_several_tokens(bits, group, add):
    """Every place of the boundary among the new tokens: also those where the ring has no room left for a launch of its own
    (the new rows take slots of the group), where two groups are completed, and more tokens than the residual."""
    for over in {0, 1, add - 1}:
        n1 = 128 + group * 9 + over
        _check(8, 2, bits, group, 128, [n1 - add], add)


@pytest.mark.parametrize("bits,group", SETTINGS)
def test_ragged_batches(bits, group):
    full = 128 + group * 12 - 1
    _check(8, 2, bits, group, 128, [full, full - 1, 0, group, 128 + group - 1, 1], 1)
    _check(8, 8, bits, group, 128, [full] * 40, 1)          # more workgroups than one round: two launches
    _check(16, 2, bits, group, 128, [128 + group * 100 - 1, full], 1)


def test_not_finite_rows():
    for bits, group in SETTINGS:
        (one, two), q, kn, vn = _pair(8, 2, bits, group, 128, 1, [128 + group * 3 - 1], 1)
        for L in (one, two):
            for name in ("k_resid", "v_resid"):
                r = L.buffers[name].view(torch.float16).view(-1, 128)
                r[7, 11], r[9, 12], r[20, 13] = float("inf"), float("nan"), -float("inf")
        one.decode(q, SM, kn, vn)
        two.append(kn, vn)
        torch.cuda.synchronize()
        _same(one, two)
