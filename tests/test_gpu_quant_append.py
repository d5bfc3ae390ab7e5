"""The append launch of a quantized layer where it can go wrong: units of two code blocks of which the
last is half empty, tokens to quantize that sit partly in the ring, ring slots that are written in the
same launch or (long appends onto a tail) only after the quantization, decision points hit exactly, flat and
tiny groups.  Bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import paper_2505_19586_amd as tkv
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


def test_ragged_batch():
    """Sequences with no group, one group and many in one launch."""
    lens = [7, 160, 161, 1000]
    shape = HeadShape(8, 2, 128)
    ins = [make_layer(m, config=2, layer=1, seq=m, shape=shape) for m in lens]
    layer = tkv.QuantLayer(n_q_heads=8, n_kv_heads=2, bits=2, capacity=1024, batch=4)
    layer.append(to_new_batch([i.k for i in ins], max(lens)), to_new_batch([i.v for i in ins], max(lens)), n_valid=lens)
    for b, i in enumerate(ins):
        check_quant_cache(layer, b, i.k, i.v)
