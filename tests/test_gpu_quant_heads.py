"""GPU tests of groups of 5 to 8 query heads per KV head (one workgroup): every head keeps a softmax reference of its
own, whatever the logits of the other heads of its group."""
import numpy as np
import pytest
import torch

import paper_2505_19586_amd as tkv
from oracle import attention
from synth import HeadShape, make_layer

from gpu_util import attn_err, check_quant_cache, to_new

pytestmark = pytest.mark.gpu
TOL = 2e-3
SM = 1.0 / np.sqrt(128.0)
SETTINGS = [(2, 32), (4, 32), (1, 64), (2, 64), (1, 32), (4, 64)]
APART = (0.25, 1.0, 4.0, 16.0, 16.0, 4.0, 1.0, 0.25)  # heads h and h + 4 a factor of 4 or 64 apart


@pytest.mark.parametrize("bits,g", SETTINGS)
@pytest.mark.parametrize("hq", [64, 56, 48, 40])
@pytest.mark.parametrize("scales", [APART, tuple(1.0 / (4 * s) for s in APART), (8.0, 8.0, 8.0, 8.0, 0.5, 0.5, 0.5, 0.5),
                                    (0.5, 0.5, 0.5, 0.5, 8.0, 8.0, 8.0, 8.0)])
def test_heads_scaled_apart(bits, g, hq, scales):
    print(f"case heads apart bits={bits} g={g} hq={hq} scales={scales}", flush=True)
    n, hkv = 3001, 8
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
def test_a_head_that_is_not_finite_stays_alone(bits, g, bad):
    n, hq, hkv = 1500, 12, 2
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
