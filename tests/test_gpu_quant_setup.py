"""Set-up of the matrix-core decode kernel where waves do different parts of it: waves with and without blocks, one or several that
work out zero-point terms (more than 16 and more than 16 per wave), new rows stored by few threads, by all and in a second round."""
import pytest
import torch

import paper_2505_19586_amd as tkv

pytestmark = pytest.mark.gpu
SM = 128 ** -0.5


@pytest.mark.parametrize("bits,g", [(2, 32), (4, 32), (1, 64), (2, 64)])
@pytest.mark.parametrize("hq,hkv", [(6, 2), (12, 2)])  # workgroups of up to four heads, of up to eight
@pytest.mark.parametrize("n,target", [(180, 0), (450, 0), (900, 0), (5000, 0), (7000, 2), (7000, 4), (15500, 4)])
def test_waves_with_different_parts(bits, g, hq, hkv, n, target):
    gen = torch.Generator(device="cuda").manual_seed(n + hq)
    k, v = (torch.randn(1, n + 80, hkv, 128, generator=gen, device="cuda").half() for _ in range(2))
    k[..., 5] += 8.0  # zero-points that matter
    q = torch.randn(1, hq, 128, generator=gen, device="cuda").half()
    one, two = (tkv.QuantLayer(n_q_heads=hq, n_kv_heads=hkv, bits=bits, group_size=g, capacity=(n + 80) // g * g + g) for _ in range(2))
    at = n
    for layer in (one, two):
        layer.append(k[:, :at].contiguous(), v[:, :at].contiguous())
    try:
        for add in (1, 16, 24, 31):  # 32 threads, 512 (all of 8 waves), 768 (all of 12), more than there are
            print(f"case setup {bits}/{g} {hq}/{hkv} n={at} add={add} target={target}", flush=True)
            kn, vn = k[:, at:at + add].contiguous(), v[:, at:at + add].contiguous()
            tkv.debug_quant_attn_config(0, target or -1)
            one.workspace[:one.desc.n_q_heads * 257 * 132 * 4].fill_(255)  # NaN in every partial
            got = one.decode(q, SM, kn, vn).float()
            two.append(kn, vn)
            tkv.debug_quant_attn_config(1)
            want = two.attn_decode(q, SM).float()
            for name in one.buffers:
                assert torch.equal(one.buffers[name], two.buffers[name]), name
            # both kernels are within 2e-3 of float64 on their own
            assert ((got - want).abs().amax(-1) <= 4e-3 * want.abs().amax(-1)).all()
            at += add
    finally:
        tkv.debug_quant_attn_config(0, -1)
