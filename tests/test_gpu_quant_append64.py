"""Groups of 64 at the rule that separates the two append kernels (one workgroup per compute unit): the same rows as few heads and
as so many that the other kernel takes them, from an empty cache, onto a tail and one token at a time, give the same bytes."""
import pytest
import torch

import paper_2505_19586_amd as tkv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("pieces", [[200], [191, 1, 130], [190, 700], [640, 63, 1]])
def test_both_kernels_write_the_same_bytes(bits, pieces):
    print(f"case append64 {bits} {pieces}", flush=True)
    n, few, many = sum(pieces), 3, 300
    gen = torch.Generator(device="cuda").manual_seed(n)
    k, v = (torch.randn(1, n, few, 128, generator=gen, device="cuda").half() for _ in range(2))
    for x in (k, v):
        for special in (float("inf"), float("nan"), 60000.0, 0.0):
            x[torch.rand(x.shape, generator=gen, device="cuda") < 0.003] = special
    layers = [tkv.QuantLayer(n_q_heads=h, n_kv_heads=h, bits=bits, group_size=64, capacity=1024) for h in (few, many)]
    at = 0
    for m in pieces:
        for layer, reps in zip(layers, (1, many // few)):
            layer.append(*(x[:, at:at + m].repeat(1, 1, reps, 1) for x in (k, v)))
        at += m
    for name in layers[0].buffers:
        a, b = (layer.buffers[name].view(layer.desc.n_kv_heads, -1) for layer in layers)
        assert torch.equal(a.repeat(many // few, 1), b), name
