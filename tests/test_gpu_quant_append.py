"""The append launch of a quantized layer where it can go wrong: units of two code blocks of which the
last is half empty, tokens to quantize that sit partly in the ring, ring slots that are written in the
same launch or (long appends onto a tail) only after the quantization, decision points hit exactly, flat and
tiny groups.  Bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import paper_2505_19586_amd as tkv
from oracle import quant
from synth import HeadShape, make_layer

from gpu_util import check_quant_cache, to_new, to_new_batch

pytestmark = pytest.mark.gpu
SETTINGS = [(1, 32), (2, 32), (4, 32), (1, 64), (2, 64), (4, 64)]


@pytest.mark.parametrize("bits,g", SETTINGS)
@pytest.mark.parametrize("pieces", [
    [193],                    # one group of 32, none of 64
    [256 + 64 * 5 + 32],      # units of 64 tokens: the last one half full with groups of 32
    [150, 1, 1, 200, 31, 33], # short appends, groups partly from the ring, slots reused in the same launch
    [190, 700],               # more new tokens than the ring holds: two launches
])
def test_append_pieces(bits, g, pieces):
    print(f"case append bits={bits} g={g} pieces={pieces}", flush=True)
    n = sum(pieces)
    shape = HeadShape(8, 2, 128)
    inp = make_layer(n, config=2, layer=0, seq=n % 61, shape=shape)
    layer = tkv.QuantLayer(n_q_heads=8, n_kv_heads=2, bits=bits, group_size=g, capacity=1024)
    kd, vd = to_new(inp.k), to_new(inp.v)
    at = 0
    for m in pieces:
        layer.append(kd[:, at:at + m].contiguous(), vd[:, at:at + m].contiguous())
        at += m
        check_quant_cache(layer, 0, inp.k[:, :at], inp.v[:, :at])


@pytest.mark.parametrize("bits,g", SETTINGS)
def test_decision_points_flat_and_tiny_groups(bits, g):
    """Values on a coarse lattice: quotients that are exactly j - 1/2 (ties to even), groups of one value
    (scaler 0), and fp16 subnormals (a scaler rounded so far that the clamp acts)."""
    print(f"case lattice bits={bits} g={g}", flush=True)
    rng = np.random.default_rng([bits, g])
    n, hkv = 512, 2
    qmax = 2 ** bits - 1
    k = rng.integers(0, 2 * qmax + 1, (hkv, n, 128)).astype(np.float16) / np.float16(2)
    v = (rng.integers(0, 12, (hkv, n, 128)) * 2.0 ** -24).astype(np.float16)
    k[0, :64] = np.float16(1.25)
    v[1, 64:128] = np.float16(-3)
    layer = tkv.QuantLayer(n_q_heads=4, n_kv_heads=hkv, bits=bits, group_size=g, capacity=n)
    layer.append(to_new(k), to_new(v))
    check_quant_cache(layer, 0, k, v)


def _eq4_with_specials(x, bits):
    """The oracle's steps where infinities and NaN occur: minimum and maximum pass NaN by, the clamp takes NaN to 0."""
    qmax = np.float32((1 << bits) - 1)
    with np.errstate(all="ignore"):
        mn, mx = np.fmin.reduce(x, axis=-1), np.fmax.reduce(x, axis=-1)
        s = ((mx.astype(np.float32) - mn.astype(np.float32)) / qmax).astype(np.float16)
        t = (x.astype(np.float32) - mn.astype(np.float32)[..., None]) / s.astype(np.float32)[..., None]
        code = np.fmin(np.fmax(np.rint(t), np.float32(0)), qmax)
    return np.where(s[..., None] == 0, 0, code).astype(np.uint8), s, mn


@pytest.mark.parametrize("bits,g", SETTINGS)
def test_infinities_and_nan(monkeypatch, bits, g):
    """Groups that hold infinities, NaN beside numbers, and ranges whose 1-bit scaler overflows fp16."""
    print(f"case specials bits={bits} g={g}", flush=True)
    monkeypatch.setattr(quant, "quantize_lastaxis", _eq4_with_specials)
    rng = np.random.default_rng([bits, g, 7])
    n, hkv = 512, 2
    k, v = (rng.standard_normal((hkv, n, 128)).astype(np.float16) for _ in range(2))
    for x in (k, v):
        for special in (np.inf, -np.inf, np.nan, 60000.0, -60000.0):
            x[rng.random(x.shape) < 0.004] = special
    layer = tkv.QuantLayer(n_q_heads=4, n_kv_heads=hkv, bits=bits, group_size=g, capacity=n)
    layer.append(to_new(k), to_new(v))
    check_quant_cache(layer, 0, k, v)


@pytest.mark.parametrize("bits,g", SETTINGS)
@pytest.mark.parametrize("steps", [
    [(129, 500)],               # up to 11 groups of 32 per sequence from an empty cache: odd and even numbers of them
    [(130, 190), (300, 700)],   # onto a tail whose ring slots are read while others are to be written
    [(500, 650), (0, 2), (40, 96)],
])
def test_many_groups(bits, g, steps):
    """Batches whose groups are more than the kernel for a few groups takes (the last step of the third case is not)."""
    print(f"case many groups bits={bits} g={g} steps={steps}", flush=True)
    batch, hkv = 64, 4
    inp = make_layer(2200, config=2, layer=1, seq=5, shape=HeadShape(8, hkv, 128))
    kd, vd = to_new(inp.k)[0], to_new(inp.v)[0]                       # sequence b: tokens 11 b and on
    layer = tkv.QuantLayer(n_q_heads=8, n_kv_heads=hkv, bits=bits, group_size=g, capacity=1024, batch=batch)
    at = np.zeros(batch, np.int64)
    for lo, hi in steps:
        add = np.array([lo + (37 * b) % (hi - lo + 1) for b in range(batch)], np.int32)
        k, v = (torch.stack([x[11 * b + at[b]:][:hi] for b in range(batch)]) for x in (kd, vd))
        layer.append(k, v, n_valid=add)
        at += add
        for b in (0, 1, 2, 13, 37, 63):
            check_quant_cache(layer, b, inp.k[:, 11 * b:11 * b + at[b]], inp.v[:, 11 * b:11 * b + at[b]])


def test_ragged_batch():
    """Sequences with no group, one group and many in one launch."""
    lens = [7, 160, 161, 1000]
    shape = HeadShape(8, 2, 128)
    ins = [make_layer(m, config=2, layer=1, seq=m, shape=shape) for m in lens]
    layer = tkv.QuantLayer(n_q_heads=8, n_kv_heads=2, bits=2, capacity=1024, batch=4)
    layer.append(to_new_batch([i.k for i in ins], max(lens)), to_new_batch([i.v for i in ins], max(lens)), n_valid=lens)
    for b, i in enumerate(ins):
        check_quant_cache(layer, b, i.k, i.v)
