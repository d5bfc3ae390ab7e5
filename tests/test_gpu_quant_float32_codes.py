"""Float32 quantized attention at the ends of the scalers' range, where codes and scalers meet scaled by powers of two: the bits of the
shape-generic reference kernel.  Every code of every place of an octet occurs; the largest scalers are near the largest that finite
keys and values yield (range over 15 at 4 bits, at most 8734; over 1 at 1 bit, near fp16's largest number, and infinity where a group
spans more than that), the smallest are subnormals."""
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


@pytest.mark.parametrize("of", ["keys", "values"])
@pytest.mark.parametrize("hq,hkv", [(2, 2), (4, 2), (8, 2)])
def test_infinite_scalers(of, hq, hkv):
    """1 bit, groups that span more than 65504: the scaler is infinite, code 0 times it is NaN, code 1 infinity.  NaN where the
    reference kernel has it (a group of values: its 32 channels; keys leave a head without weights), else its bits."""
    n = 1500
    print(f"case f32 infinite {of} {hq}/{hkv}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(hq)
    k, v = (torch.randn(1, n, hkv, 128, generator=gen, device="cuda").half() for _ in range(2))
    x = k if of == "keys" else v
    x[0, 300, 1, 40], x[0, 301, 1, 40] = 60000.0, -60000.0  # a channel's group of 32 tokens (288 to 319)
    x[0, 700, 1, 64], x[0, 700, 1, 90] = -50000.0, 50000.0  # a token's group of 32 channels (64 to 95)
    q = torch.randn(1, hq, 128, generator=gen, device="cuda").half()
    layer = tkv.QuantLayer(n_q_heads=hq, n_kv_heads=hkv, bits=1, group_size=32, capacity=1536)
    layer.append(k, v)
    assert torch.isinf(layer.view("k_scale" if of == "keys" else "v_scale")).any()
    try:
        tkv.debug_quant_attn_config(1)
        want = layer.attn_decode(q, SM).clone()
    finally:
        tkv.debug_quant_attn_config(0)
    got = layer.attn_decode(q, SM)
    assert torch.isfinite(want[:, :hq // 2]).all() and (of == "keys" or torch.isnan(want[:, hq // 2:]).any())
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    finite = ~torch.isnan(want)
    assert torch.equal(got[finite].view(torch.int16), want[finite].view(torch.int16))
