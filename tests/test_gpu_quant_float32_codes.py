"""Float32 quantized attention at the ends of the scalers' range, where codes and scalers meet scaled by powers of two: the bits of the
shape-generic reference kernel.  Every code of every place of an octet occurs; the largest scalers are near fp16's largest
number, the smallest are subnormals."""
import pytest
import torch

import paper_2505_19586_amd as tkv

pytestmark = pytest.mark.gpu
SM = 128 ** -0.5


@pytest.mark.parametrize("bits,g", [(4, 64), (1, 32)])
@pytest.mark.parametrize("hq,hkv", [(2, 2), (4, 2), (8, 2)])  # one, two and four heads per workgroup
@pytest.mark.parametrize("k_max,v_max", [(1.0, 32000.0), (32000.0, 1.0), (2.0 ** -20, 2.0 ** -14), (2.0 ** -14, 2.0 ** -18)])
def test_scaler_range(bits, g, hq, hkv, k_max, v_max):
    n = 1500
    print(f"case f32 codes {bits}/{g} {hq}/{hkv} {k_max} {v_max}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(int(hq))
    k, v = ((m * (2.0 * torch.rand(1, n, hkv, 128, generator=gen, device="cuda") - 1.0)).half() for m in (k_max, v_max))
    q = (torch.randn(1, hq, 128, generator=gen, device="cuda") / max(k_max, 1.0)).half()
    layer = tkv.QuantLayer(n_q_heads=hq, n_kv_heads=hkv, bits=bits, group_size=g, capacity=1536)
    layer.append(k, v)
    try:
        tkv.debug_quant_attn_config(1)
        want = layer.attn_decode(q, SM).clone()
    finally:
        tkv.debug_quant_attn_config(0)
    assert torch.isfinite(want).all() and want.abs().max() > 0
    assert torch.equal(layer.attn_decode(q, SM).view(torch.int16), want.view(torch.int16))
