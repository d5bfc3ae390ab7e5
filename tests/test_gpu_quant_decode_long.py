"""tkv_quant_decode beyond the longest cache of the matrix-core kernel (256 chunks of 512 blocks of 32 tokens): the step is the append
and the attention one after the other, whether it completes a quantization group or not."""
import pytest
import torch

import paper_2505_19586_amd as tkv

pytestmark = pytest.mark.gpu


def test_steps_of_a_cache_of_more_than_4_mi_tokens():
    n, piece, group = 4194304 + 64 * 40 + 61, 1 << 18, 64  # the third of these steps completes a group
    gen = torch.Generator(device="cuda").manual_seed(4)
    one, two = (tkv.QuantLayer(n_q_heads=1, n_kv_heads=1, bits=1, group_size=group, residual=128, capacity=n + 67) for _ in range(2))
    for a in range(0, n, piece):
        k, v = (torch.randn(1, min(piece, n - a), 1, 128, generator=gen, device="cuda").half() for _ in range(2))
        for layer in (one, two):
            layer.append(k, v)
    for step in range(4):
        print(f"case long step {step}", flush=True)
        kn, vn, q = (torch.randn(1, 1, 1, 128, generator=gen, device="cuda").half() for _ in range(3))
        got = one.decode(q[:, 0], 128 ** -0.5, kn, vn)
        two.append(kn, vn)
        want = two.attn_decode(q[:, 0], 128 ** -0.5)
        assert list(one.seq_len) == list(two.seq_len) == [n + step + 1]
        assert torch.isfinite(got).all() and torch.equal(got.view(torch.int16), want.view(torch.int16))
    for name in one.buffers:
        assert torch.equal(one.buffers[name].view(torch.uint8), two.buffers[name].view(torch.uint8)), name
