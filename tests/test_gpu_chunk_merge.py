"""Merge of a sequence's split-K chunks by its last workgroup at the edges of what a wave takes: one to eight query heads, two to
256 chunks, stale partials in the scratch memory."""
import pytest
import torch

import paper_2505_19586_amd as tkv

pytestmark = pytest.mark.gpu
SM = 128 ** -0.5


@pytest.mark.parametrize("bits,g", [(2, 32), (4, 32), (1, 64)])
@pytest.mark.parametrize("hq", [1, 3, 4, 5, 6, 8])
def test_chunk_counts(bits, g, hq):
    n = 32768 + 165  # blocks of 32: 1024, at least one per wave and chunk
    gen = torch.Generator(device="cuda").manual_seed(hq)
    k, v = (torch.randn(1, n, 1, 128, generator=gen, device="cuda").half() for _ in range(2))
    q = 2.0 * torch.randn(1, hq, 128, generator=gen, device="cuda").half()
    layer = tkv.QuantLayer(n_q_heads=hq, n_kv_heads=1, bits=bits, group_size=g, capacity=n + g - n % g)
    layer.append(k, v)
    try:
        tkv.debug_quant_attn_config(1)
        want = layer.attn_decode(q, SM).float()
        for target in (2, 3, 7, 21, 22, 23, 63, 64, 65, 66, 67, 85, 128, 129, 256):
            print(f"case merge {bits}/{g} heads={hq} chunks={target}", flush=True)
            tkv.debug_quant_attn_config(0, target)
            layer.workspace[:hq * 257 * 132 * 4].fill_(255)  # NaN in every partial
            got = layer.attn_decode(q, SM).float()
            # both kernels are within 2e-3 of float64 on their own
            assert ((got - want).abs().amax(-1) <= 4e-3 * want.abs().amax(-1)).all(), target
    finally:
        tkv.debug_quant_attn_config(0, -1)
