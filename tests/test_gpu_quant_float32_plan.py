"""Float32 quantized attention where the plan of its chunks turns: the longest short chunks and the shortest long ones (tails in front
of them or behind), as many workgroups as four per compute unit and one more chunk.  The bits of the shape-generic reference kernel."""
import pytest
import torch

import paper_2505_19586_amd as tkv

pytestmark = pytest.mark.gpu
SM = 128 ** -0.5


@pytest.mark.parametrize("bits,g", [(4, 64), (1, 32)])
@pytest.mark.parametrize("hq,hkv,batch,lens", [
    # blocks per chunk in the order of the lengths: 5 to 12, 9 and 10, 8 to 11, one chunk of 5 to 11
    (16, 8, 24, (750, 900, 1100, 1300, 1500)), (8, 8, 6, (5500, 6000, 6500)), (12, 4, 24, (2500, 3000)), (32, 32, 16, (300, 400, 500))])
def test_bits_of_the_reference_kernel(bits, g, hq, hkv, batch, lens):
    gen = torch.Generator(device="cuda").manual_seed(batch)
    k, v = (torch.randn(batch, max(lens), hkv, 128, generator=gen, device="cuda").half() for _ in range(2))
    q = 2.0 * torch.randn(batch, hq, 128, generator=gen, device="cuda").half()
    layer = tkv.QuantLayer(n_q_heads=hq, n_kv_heads=hkv, bits=bits, group_size=g, capacity=(max(lens) + g) // g * g, batch=batch)
    at = 0
    for n in lens:
        print(f"case f32 plan bits={bits} {hq}/{hkv} B={batch} n={n}", flush=True)
        layer.append(k[:, at:n].contiguous(), v[:, at:n].contiguous())
        at = n
        layer.workspace[:batch * hq * 257 * 132 * 4].fill_(255)  # NaN in every partial
        got = layer.attn_decode(q, SM).clone()
        try:
            tkv.debug_quant_attn_config(1)
            want = layer.attn_decode(q, SM).clone()
        finally:
            tkv.debug_quant_attn_config(0)
        assert torch.isfinite(got).all()
        assert torch.equal(got.view(torch.int16), want.view(torch.int16))
