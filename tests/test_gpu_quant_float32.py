"""GPU tests of the settings that stay in float32 (4 bits with groups of 64, 1 bit with groups of 32): bit for bit the
shape-generic reference kernel's results, the same on every call, over the whole fp16 input range."""
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
SETTINGS = [(4, 64), (1, 32)]


def reference(call):
    try:
        tkv.debug_quant_attn_config(1)
        return call().clone()
    finally:
        tkv.debug_quant_attn_config(0)


def same_bits(a, b):
    return torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("bits,g", SETTINGS)
@pytest.mark.parametrize("heads", [(8, 8), (16, 8), (6, 2), (32, 8), (10, 2), (64, 8)])  # groups of 1, 2, 3, 4, 5, 8
@pytest.mark.parametrize("lens,residual", [
    ([1], 128), ([31], 64), ([191], 64), ([192], 128),       # the tail alone; the first blocks
    ([5000], 128),                                           # a few blocks per stream, ring wrapped
    ([70001], 192),                                           # many chunks; an odd number of tail pieces
    ([2500, 0, 130, 4097, 1024], 128),                       # chunks past the end of the shorter sequences
])
def test_bits_of_the_reference_kernel(bits, g, heads, lens, residual):
    print(f"case f32 bits={bits} g={g} heads={heads} lens={lens} W={residual}", flush=True)
    hq, hkv = heads
    gen = torch.Generator(device="cuda").manual_seed(len(lens) * 100 + hq)
    n = max(lens)
    k, v = (torch.randn(len(lens), n, hkv, 128, generator=gen, device="cuda").half() for _ in range(2))
    k *= 1.0 + 4.0 * (torch.rand(hkv, 128, generator=gen, device="cuda") > 0.9)
    v[:, ::7] *= 1e-4                                        # scalers in fp16's subnormals
    v[:, ::11] *= 600.0
    q = torch.randn(len(lens), hq, 128, generator=gen, device="cuda").half()
    q *= (2.0 ** (torch.arange(hq, device="cuda") % 7 - 2))[:, None]
    layer = tkv.QuantLayer(n_q_heads=hq, n_kv_heads=hkv, bits=bits, group_size=g, residual=residual,
                           capacity=(n + g) // g * g, batch=len(lens))
    layer.append(k, v, n_valid=np.array(lens, np.int32))
    want = reference(lambda: layer.attn_decode(q, SM))
    for _ in range(2):
        assert same_bits(layer.attn_decode(q, SM), want)
    if len(lens) * hq < 64:                                  # (what the fixed scratch memory takes for sure)
        assert same_bits(layer.attn_decode_static(q, SM, torch.empty_like(q)), want)
    odd = torch.empty(q.numel() + 1, dtype=torch.float16, device="cuda")[1:].view_as(q).copy_(q)
    assert odd.data_ptr() % 4 == 2
    assert same_bits(layer.attn_decode(odd, SM), want)


def test_fixed_scratch_memory_of_a_large_batch():
    """63 sequences of 32 query heads: the usual three chunks and the tail make more partials than the fixed array
    holds, two chunks do not.  Float32 sums in another order: the results differ by their fp16 rounding at most."""
    gen = torch.Generator(device="cuda").manual_seed(5)
    k, v = (torch.randn(63, 700, 8, 128, generator=gen, device="cuda").half() for _ in range(2))
    q = torch.randn(63, 32, 128, generator=gen, device="cuda").half()
    layer = tkv.QuantLayer(n_q_heads=32, n_kv_heads=8, bits=4, group_size=64, capacity=704, batch=63)
    layer.append(k, v)
    want = layer.attn_decode(q, SM)
    got = layer.attn_decode_static(q, SM, torch.empty_like(q))
    assert attn_err(got, want.float().cpu().numpy().astype(np.float64)) <= 2.0 ** -10


@pytest.mark.parametrize("bits,g", SETTINGS)
def test_decode_step_is_append_and_attention(bits, g):
    """tkv_quant_decode over steps with and without a completed group: the bits of the two calls."""
    lens = [1000, 447]
    inps = [make_layer(n + 70, seq=60 + b) for b, n in enumerate(lens)]
    one, two = (tkv.QuantLayer(bits=bits, group_size=g, capacity=1088, batch=2) for _ in range(2))
    for layer in (one, two):
        layer.append(to_new_batch([i.k[:, :n] for i, n in zip(inps, lens)], 1000),
                     to_new_batch([i.v[:, :n] for i, n in zip(inps, lens)], 1000), n_valid=lens)
    q = torch.from_numpy(np.stack([i.q for i in inps])).cuda()
    for step in range(70):
        kn, vn = (to_new_batch([x[:, n + step:n + step + 1] for x, n in zip(xs, lens)], 1)
                  for xs in ([i.k for i in inps], [i.v for i in inps]))
        out = one.decode(q, SM, kn, vn).clone()
        two.append(kn, vn)
        assert same_bits(out, reference(lambda: two.attn_decode(q, SM))), step


@pytest.mark.parametrize("bits,g", SETTINGS)
@pytest.mark.parametrize("k_scale,q_scale,v_scale", [(64.0, 64.0, 1.0), (1.0, 1.0, 4000.0), (1.0, 1.0, 1e-2)])
def test_input_range(bits, g, k_scale, q_scale, v_scale):
    """Query-times-scaler products and value scalers past fp16's range, and small values: float32 has none of the matrix
    cores' limits.  Bound, relative to the head's largest output: its fp16 rounding (spacing 2^-24 below 2^-14), float32
    sums (1e-5) and the weights' share of the logits' rounding, 128 2^-24 |q|.|k-hat| (one token holds all the weight
    where that is large)."""
    inp = make_layer(3000, seq=9, shape=HeadShape(32, 8, 128))
    k, v, q = ((x.astype(np.float32) * s).astype(np.float16) for x, s in ((inp.k, k_scale), (inp.v, v_scale), (inp.q, q_scale)))
    k[:, :2800] *= np.linspace(0.2, 1.0, 2800, dtype=np.float32).astype(np.float16)[:, None]  # logits that rise over the sequence
    layer = tkv.QuantLayer(bits=bits, group_size=g, capacity=3072)
    layer.append(to_new(k), to_new(v))
    ref = check_quant_cache(layer, 0, k, v)
    out = layer.attn_decode(torch.from_numpy(q)[None].cuda(), SM)
    assert torch.isfinite(out).all()
    want = attention.quant_attention(q, ref, SM)
    largest = np.abs(want).max(axis=-1).min()
    assert attn_err(out[0], want) <= 2.0 ** -11 + 2.0 ** -25 / largest + 1e-5 + logit_share(q, ref, want)


def logit_share(q, ref, want):
    """Largest change of a head's output, relative to its largest element, when every logit is off by its float32
    rounding bound the other way than the rest: twice the sum of w (1 - w) |error|, times the largest |v - out|."""
    kh = np.concatenate([quant.dequantize_k(ref), ref.k_resid.astype(np.float64)], axis=1)
    vh = np.concatenate([quant.dequantize_v(ref), ref.v_resid.astype(np.float64)], axis=1)
    worst = 0.0
    for i in range(q.shape[0]):
        h = i // (q.shape[0] // kh.shape[0])
        qi = q[i].astype(np.float64)
        lg = kh[h] @ qi * SM
        err = 3 * 2.0 ** -24 * np.sqrt(128) * np.sqrt((kh[h] ** 2) @ (qi ** 2)) * SM
        w = np.exp(lg - lg.max())
        w /= w.sum()
        worst = max(worst, (w * (1 - w) * err).sum() * 2 * np.abs(vh[h] - want[i]).max() / np.abs(want[i]).max())
    return worst
