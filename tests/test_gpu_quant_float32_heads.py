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


@pytest.mark.parametrize("bits,g", [(4, 64), (1, 32)])
@pytest.mark.parametrize("hq,hkv,batch,lens", [
    # tails counted: (sequences, KV heads, groups of 1 head) x (chunks + 2) <= 1056, (... of 2 heads) x (chunks + 1) <= 1056 or not
    (32, 8, 10, (230,)), (32, 8, 11, (230,)), (32, 8, 32, (150, 300, 430)), (32, 8, 34, (230,)), (24, 8, 16, (230, 300)), (16, 8, 21, (230,)),
    (16, 8, 23, (230,)), (16, 8, 40, (170,)), (64, 8, 16, (170, 300, 1087)), (12, 2, 64, (300,))])
def test_bits_of_the_reference_kernel_many_short_sequences(bits, g, hq, hkv, batch, lens):
    gen = torch.Generator(device="cuda").manual_seed(batch)
    k, v = (torch.randn(batch, max(lens), hkv, 128, generator=gen, device="cuda").half() for _ in range(2))
    q = 2.0 * torch.randn(batch, hq, 128, generator=gen, device="cuda").half()
    layer = tkv.QuantLayer(n_q_heads=hq, n_kv_heads=hkv, bits=bits, group_size=g, residual=128, capacity=(max(lens) + g) // g * g,
                           batch=batch)
    at = 0
    for n in lens:
        print(f"case f32 short bits={bits} {hq}/{hkv} B={batch} n={n}", flush=True)
        layer.append(k[:, at:n].contiguous(), v[:, at:n].contiguous())
        at = n
        got = layer.attn_decode(q, SM).clone()
        try:
            tkv.debug_quant_attn_config(1)
            want = layer.attn_decode(q, SM).clone()
        finally:
            tkv.debug_quant_attn_config(0)
        assert torch.equal(got.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("bits,g", [(4, 64), (1, 32)])
@pytest.mark.parametrize("hq,hkv,lens", [(8, 8, (1, 700, 150)), (32, 8, (0, 5000, 4223)), (21, 7, (250, 249, 60000)),
                                         (40, 5, (95, 96, 12000))])
def test_decode_steps_join_the_ring_in_the_attention(bits, g, hq, hkv, lens):
    """Several new tokens at once, none for some sequences, the ring's end, steps that complete a group: cache and output of
    the append and the attention one after the other."""
    gen = torch.Generator(device="cuda").manual_seed(hq)
    cap = (max(lens) + 400) // g * g
    one, two = (tkv.QuantLayer(n_q_heads=hq, n_kv_heads=hkv, bits=bits, group_size=g, residual=64, capacity=cap, batch=3)
                for _ in range(2))
    k, v = (torch.randn(3, max(lens), hkv, 128, generator=gen, device="cuda").half() for _ in range(2))
    for layer in (one, two):
        layer.append(k, v, n_valid=list(lens))
    for step, (n_new, n_valid) in enumerate([(1, None), (3, (3, 0, 2)), (1, (0, 0, 0)), (33, (33, 1, 20)), (1, None), (17, None), (20, None)]):
        print(f"case f32 ring bits={bits} {hq}/{hkv} lens={lens} step={step}", flush=True)
        kn, vn = (torch.randn(3 * n_new * hkv * 128 + 1, generator=gen, device="cuda").half()[1:].view(3, n_new, hkv, 128)
                  for _ in range(2))  # (rows at odd fp16 addresses)
        q = torch.randn(3, hq, 128, generator=gen, device="cuda").half()
        got = one.decode(q, SM, kn, vn, n_valid=n_valid).clone()
        two.append(kn, vn, n_valid=n_valid)
        want = two.attn_decode(q, SM)
        assert torch.equal(got.view(torch.int16), want.view(torch.int16))
        assert list(one.seq_len) == list(two.seq_len)
        for name in one.buffers:
            assert torch.equal(one.buffers[name].view(torch.uint8), two.buffers[name].view(torch.uint8)), name
