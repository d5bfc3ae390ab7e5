"""Merge of a sequence's split-K chunks by its last workgroup at the edges of what a wave takes, stale partials in the scratch memory.
test_chunk_counts: one to eight query heads; up to four of them two to 87 chunks (130 at 4 bits), five to eight up to 23 in one
workgroup and 32 and more in two.  test_many_chunks: 64 to 256 chunks, five and eight heads in one workgroup."""
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


@pytest.mark.parametrize("bits,g", [(2, 32), (4, 32), (1, 64)])
@pytest.mark.parametrize("hq,n", [(1, 120000), (4, 120000), (5, 400000), (8, 400000)])
def test_many_chunks(bits, g, hq, n):
    """Second rounds of loads (beyond 64 and 66 chunks) and of weights (64, 128 and 192).  Long enough for a block per wave in
    each of 256 chunks, and that a group of five or eight heads stays one workgroup's (40 blocks per workgroup)."""
    gen = torch.Generator(device="cuda").manual_seed(hq)
    k, v = (torch.randn(1, n, 1, 128, generator=gen, device="cuda").half() for _ in range(2))
    q = 2.0 * torch.randn(1, hq, 128, generator=gen, device="cuda").half()
    layer = tkv.QuantLayer(n_q_heads=hq, n_kv_heads=1, bits=bits, group_size=g, capacity=n + g - n % g)
    layer.append(k, v)
    room = layer.workspace[:hq * 257 * 132 * 4].view(torch.float32)
    try:
        tkv.debug_quant_attn_config(1)
        want = layer.attn_decode(q, SM).float()
        for target in (64, 65, 66, 67, 128, 129, 192, 193, 256):
            print(f"case merge {bits}/{g} heads={hq} n={n} chunks={target}", flush=True)
            tkv.debug_quant_attn_config(0, target)
            room.fill_(float("nan"))
            got = layer.attn_decode(q, SM).float()
            assert int((~torch.isnan(room)).sum()) == hq * target * 130  # a sum of 128 channels, a maximum and a sum of weights each
            # both kernels are within 2e-3 of float64 on their own
            assert ((got - want).abs().amax(-1) <= 4e-3 * want.abs().amax(-1)).all(), target
    finally:
        tkv.debug_quant_attn_config(0, -1)
