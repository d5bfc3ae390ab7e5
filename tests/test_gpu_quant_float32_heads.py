"""Float32 quantized attention on both sides of the lengths at which a workgroup takes one, two or four query heads, and tails
of 1 to residual + group - 1 tokens at every place of the ring: bit for bit the shape-generic reference kernel's results."""
import pytest
import torch

import paper_2505_19586_amd as tkv

pytestmark = pytest.mark.gpu
SM = 128 ** -0.5


@pytest.mark.parametrize("bits,g", [(4, 64), (1, 32)])
@pytest.mark.parametrize("hq,hkv,lens", [
    # blocks of 32 quantized tokens / 4 = chunks; (chunks) x (sequences, KV heads, groups of 1, 2, 4 heads) <= 1024 or not
    (32, 8, (4095, 4159, 4223, 4287, 4415)), (32, 8, (8191, 8319, 8383, 8511)), (6, 2, (21800, 22100, 32700, 33100)),
    (40, 8, (3400, 3600, 5400, 5700)), (16, 8, (8191, 8319, 8383)),
    (8, 1, tuple(range(127, 200, 8)) + tuple(range(319, 400, 16)))])
def test_bits_of_the_reference_kernel(bits, g, hq, hkv, lens):
    gen = torch.Generator(device="cuda").manual_seed(hq)
    k, v = (torch.randn(1, max(lens), hkv, 128, generator=gen, device="cuda").half() for _ in range(2))
    q = 2.0 * torch.randn(1, hq, 128, generator=gen, device="cuda").half()
    layer = tkv.QuantLayer(n_q_heads=hq, n_kv_heads=hkv, bits=bits, group_size=g, residual=128, capacity=(max(lens) + g) // g * g)
    at = 0
    for n in lens:
        print(f"case f32 heads bits={bits} {hq}/{hkv} n={n}", flush=True)
        layer.append(k[:, at:n].contiguous(), v[:, at:n].contiguous())
        at = n
        got = layer.attn_decode(q, SM).clone()
        try:
            tkv.debug_quant_attn_config(1)
            want = layer.attn_decode(q, SM).clone()
        finally:
            tkv.debug_quant_attn_config(0)
        assert torch.equal(got.view(torch.int16), want.view(torch.int16))
