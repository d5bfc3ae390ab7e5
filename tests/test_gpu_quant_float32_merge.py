"""Merge of the float32 attention's parts at the edges of what a thread takes: two to 257 parts of one query head, all scratch memory
NaN before the call, against the oracle."""
import numpy as np
import pytest
import torch

import paper_2505_19586_amd as tkv
from oracle import attention
from synth import HeadShape, make_layer

from gpu_util import attn_err, check_quant_cache, to_new

pytestmark = pytest.mark.gpu
SM = 1.0 / np.sqrt(128.0)


@pytest.mark.parametrize("bits,g", [(4, 64), (1, 32)])
@pytest.mark.parametrize("parts", [2, 3, 4, 5, 7, 8, 15, 16, 17, 18, 63, 64, 65, 66, 128, 129, 130, 257])
def test_parts(bits, g, parts):
    n = 128 + 128 * (parts - 1) + 5  # one KV head: a chunk per four blocks of 32 quantized tokens, and the tail
    print(f"case f32 merge {bits}/{g} parts={parts}", flush=True)
    inp = make_layer(n, config=3, layer=1, seq=parts, shape=HeadShape(3, 1, 128))
    layer = tkv.QuantLayer(n_q_heads=3, n_kv_heads=1, bits=bits, group_size=g, capacity=n + g - n % g)
    layer.append(to_new(inp.k), to_new(inp.v))
    room = layer.workspace[:3 * 257 * 132 * 4].view(torch.float32).view(-1, 132)
    room.fill_(float("nan"))
    out = layer.attn_decode(torch.from_numpy(inp.q)[None].cuda(), SM)
    assert torch.isfinite(room[:3 * parts, 4:]).all() and torch.isnan(room[3 * parts:]).all()  # so many parts
    want = attention.quant_attention(inp.q, check_quant_cache(layer, 0, inp.k, inp.v), SM)
    err = attn_err(out[0], want)
    print(f"   err {err:.3e}", flush=True)
    # the output's rounding to fp16, at most 2^-11 of a head's largest element, and float32 sums over at most 33000 tokens
    assert err <= 2.0 ** -11 + 1e-4
