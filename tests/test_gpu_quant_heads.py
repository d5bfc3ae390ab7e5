"""GPU tests of groups of 5 to 8 query heads per KV head, served by one workgroup or by two: every head keeps a softmax
reference of its own, whatever the logits of the other heads of its group."""
import numpy as np
import pytest
import torch

import paper_2505_19586_amd as tkv
from oracle import attention, quant
from synth import HeadShape, make_layer

from gpu_util import attn_err, check_quant_cache, to_new, to_new_batch

pytestmark = pytest.mark.gpu
TOL = 2e-3
SM = 1.0 / np.sqrt(128.0)
SETTINGS = [(2, 32), (4, 32), (1, 64), (2, 64), (1, 32), (4, 64)]
APART = (0.25, 1.0, 4.0, 16.0, 16.0, 4.0, 1.0, 0.25)  # heads h and h + 4 a factor of 4 or 64 apart


@pytest.fixture(params=["two workgroups", "one workgroup"])
def route(request):
    """Sequences as short as these are served by two workgroups per KV head and chunk.  One workgroup is what a launch
    has that aims at few: one per KV head and 2000 tokens makes the 80 blocks or more from which that is taken."""
    def choose(hkv, n):
        if request.param == "one workgroup":
            tkv.debug_quant_attn_config(0, hkv * max(1, n // 2000))
    yield choose
    tkv.debug_quant_attn_config(0, -1)


@pytest.mark.parametrize("bits,g", SETTINGS)
@pytest.mark.parametrize("hq", [64, 56, 48, 40])
@pytest.mark.parametrize("scales", [APART, tuple(1.0 / (4 * s) for s in APART), (8.0, 8.0, 8.0, 8.0, 0.5, 0.5, 0.5, 0.5),
                                    (0.5, 0.5, 0.5, 0.5, 8.0, 8.0, 8.0, 8.0)])
def test_heads_scaled_apart(bits, g, hq, scales, route):
    print(f"case heads apart bits={bits} g={g} hq={hq} scales={scales}", flush=True)
    n, hkv = 3001, 8
    route(hkv, n)
    inp = make_layer(n, shape=HeadShape(hq, hkv, 128), seq=17)
    q = inp.q * np.tile(np.array(scales[:hq // hkv], np.float16), hkv)[:, None]
    layer = tkv.QuantLayer(n_q_heads=hq, n_kv_heads=hkv, bits=bits, group_size=g, capacity=3072)
    layer.append(to_new(inp.k), to_new(inp.v))
    ref = check_quant_cache(layer, 0, inp.k, inp.v)
    out = layer.attn_decode(torch.from_numpy(q)[None].cuda(), SM)
    err = attn_err(out[0], attention.quant_attention(q, ref, SM))
    print(f"   err {err:.3e}", flush=True)
    assert err <= TOL


@pytest.mark.parametrize("bits,g", SETTINGS)
@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_a_head_that_is_not_finite_stays_alone(bits, g, bad, route):
    n, hq, hkv = 1500, 12, 2
    route(hkv, n)
    inp = make_layer(n, shape=HeadShape(hq, hkv, 128), seq=18)
    layer = tkv.QuantLayer(n_q_heads=hq, n_kv_heads=hkv, bits=bits, group_size=g, capacity=1536)
    layer.append(to_new(inp.k), to_new(inp.v))
    ref = check_quant_cache(layer, 0, inp.k, inp.v)
    want = attention.quant_attention(inp.q, ref, SM)
    q = inp.q.copy()
    q[0, 3] = q[7, 5] = bad
    out = layer.attn_decode(torch.from_numpy(q)[None].cuda(), SM)[0]
    rest = [i for i in range(hq) if i not in (0, 7)]
    assert attn_err(out[rest], want[rest]) <= TOL


@pytest.mark.parametrize("bits,g", SETTINGS)
@pytest.mark.parametrize("heads,lens,n_new", [
    ((64, 8), [2500], 1), ((40, 8), [9000], 5), ((12, 2), [4001, 130, 2600], 1), ((7, 1), [159], 3), ((8, 1), [20000], 1),
])
def test_decode_step(bits, g, heads, lens, n_new, route):
    """The step's new tokens come from the caller's buffers and end up in the ring once, whoever copies them."""
    print(f"case heads step bits={bits} g={g} heads={heads} lens={lens} new={n_new}", flush=True)
    hq, hkv = heads
    route(hkv, sum(lens))
    inps = [make_layer(n, config=3, layer=1, seq=n % 89, shape=HeadShape(hq, hkv, 128)) for n in lens]
    layer = tkv.QuantLayer(n_q_heads=hq, n_kv_heads=hkv, bits=bits, group_size=g, capacity=(max(lens) + g) // g * g, batch=len(lens))
    old = np.array(lens, np.int32) - n_new
    layer.append(to_new_batch([i.k[:, :m] for i, m in zip(inps, old)], max(old)),
                 to_new_batch([i.v[:, :m] for i, m in zip(inps, old)], max(old)), n_valid=old)
    out = layer.decode(torch.from_numpy(np.stack([i.q for i in inps])).cuda(), SM,
                       to_new_batch([i.k[:, m:] for i, m in zip(inps, old)], n_new),
                       to_new_batch([i.v[:, m:] for i, m in zip(inps, old)], n_new))
    for b, i in enumerate(inps):
        ref = check_quant_cache(layer, b, i.k, i.v)
        assert attn_err(out[b], attention.quant_attention(i.q, ref, SM)) <= TOL


@pytest.mark.parametrize("bits,g", [(2, 32), (4, 32), (1, 64), (2, 64)])
@pytest.mark.parametrize("batch", [32, 33])
def test_many_short_sequences(bits, g, batch):
    """32 sequences of 4 KV heads take 256 workgroups in two per group, 33 are served by one each."""
    n = 300
    inps = [make_layer(n - 7 * (b % 5), config=3, layer=1, seq=b, shape=HeadShape(32, 4, 128)) for b in range(batch)]
    layer = tkv.QuantLayer(n_q_heads=32, n_kv_heads=4, bits=bits, group_size=g, capacity=320, batch=batch)
    layer.append(to_new_batch([i.k for i in inps], n), to_new_batch([i.v for i in inps], n), n_valid=[i.k.shape[1] for i in inps])
    out = layer.attn_decode(torch.from_numpy(np.stack([i.q for i in inps])).cuda(), SM)
    for b in range(0, batch, 4):
        ref = check_quant_cache(layer, b, inps[b].k, inps[b].v)
        assert attn_err(out[b], attention.quant_attention(inps[b].q, ref, SM)) <= TOL


@pytest.mark.parametrize("bits,g", [(2, 32), (4, 32), (1, 64), (2, 64)])
@pytest.mark.parametrize("k_scale,q_scale,v_scale", [(64.0, 1.0, 1.0), (1.0, 64.0, 1.0), (1.0, 1.0, 100.0)])
def test_large_magnitudes(bits, g, k_scale, q_scale, v_scale, route):
    """Large key scalers, queries and values stay inside fp16 on their way to the matrix cores."""
    n, hq, hkv = 3000, 64, 8
    route(hkv, n)
    inp = make_layer(n, shape=HeadShape(hq, hkv, 128), seq=9)
    k, v, q = ((x.astype(np.float32) * s).astype(np.float16) for x, s in ((inp.k, k_scale), (inp.v, v_scale), (inp.q, q_scale)))
    layer = tkv.QuantLayer(n_q_heads=hq, n_kv_heads=hkv, bits=bits, group_size=g, capacity=3072)
    layer.append(to_new(k), to_new(v))
    ref = check_quant_cache(layer, 0, k, v)
    out = layer.attn_decode(torch.from_numpy(q)[None].cuda(), SM)[0]
    assert torch.isfinite(out).all()
    want = attention.quant_attention(q, ref, SM)
    share = logit_share(q, ref, want)
    for i in range(hq):
        assert attn_err(out[i:i + 1], want[i:i + 1]) <= TOL + share[i], i


def logit_share(q, ref, want):
    """Per head: the change of its output, relative to its largest element, when every logit is off by its rounding
    the other way than the rest.  Rounding of a logit: 2^-22 of the sum of its terms' magnitudes for the query-times-scaler
    operand in fp16 hi + lo parts, as much again for the float32 sums (scaler and zero-point terms apart)."""
    kh = np.concatenate([quant.dequantize_k(ref), ref.k_resid.astype(np.float64)], axis=1)
    vh = np.concatenate([quant.dequantize_v(ref), ref.v_resid.astype(np.float64)], axis=1)
    zero = np.zeros_like(kh)
    zero[:, :ref.n_quant] = np.repeat(ref.k_zero.astype(np.float64), ref.group, axis=1)
    out = []
    for i in range(q.shape[0]):
        h = i // (q.shape[0] // kh.shape[0])
        qi = q[i].astype(np.float64)
        err = 2.0 ** -21 * ((np.abs(kh[h] - zero[h]) + np.abs(zero[h])) @ np.abs(qi)) * SM
        lg = kh[h] @ qi * SM
        w = np.exp(lg - lg.max())
        w /= w.sum()
        out.append((w * (1 - w) * err).sum() * 2 * np.abs(vh[h] - want[i]).max() / np.abs(want[i]).max())
    return out
