"""The fp16 tail of a quantized layer (pieces of 32 tokens on the matrix cores, new tokens read from the
caller's buffers) and the split of short sequences into one or more workgroups, against the oracle."""
import numpy as np
import pytest
import torch

import paper_2505_19586_amd as tkv
from oracle import attention
from synth import HeadShape, make_layer
from synth.device import make_layer_device

from gpu_util import attn_err, check_quant_cache, to_new

pytestmark = pytest.mark.gpu
SM = 1.0 / np.sqrt(128.0)
TOL = 2e-3
# nothing quantized: what is left of the error is the fp16 rounding of the output (2^-11 of an
# element, so at most 2^-11 of a head's largest) and float32 sums over at most 1023 tokens
TOL_TAIL = 2.0 ** -11 + 1e-4


@pytest.mark.parametrize("bits,g,residual,n,n_new,heads", [
    (2, 32, 128, 1, 1, (32, 8)),        # a single token, from the call itself
    (2, 32, 128, 8, 8, (32, 8)),        # all tokens are new
    (2, 32, 128, 33, 1, (16, 2)),       # second piece of one token
    (2, 32, 128, 159, 8, (3, 1)),       # nothing quantized, last piece one short of full
    (4, 32, 992, 1023, 3, (32, 8)),     # 32 pieces: four per wave of 8
    (1, 64, 960, 1023, 1, (8, 8)),      # one query head per KV head, three pieces per wave of 12
    (2, 64, 128, 191, 5, (64, 8)),      # 8 query heads
    (2, 32, 992, 1020, 5, (40, 8)),     # 5 query heads, three pieces per wave of 12
    (2, 32, 128, 896, 1, (32, 8)),      # 24 blocks and 4 pieces: the longest that one workgroup sweeps
    (2, 32, 128, 897, 1, (32, 8)),      # past it: several, merged
    (4, 32, 128, 512, 1, (32, 8)),      # the same line for workgroups of 8 waves
    (4, 32, 128, 513, 2, (32, 8)),
    (2, 32, 256, 5000, 1, (10, 2)),     # nine pieces behind many blocks, ring wrapped
    (1, 64, 128, 3010, 7, (28, 4)),
    (2, 32, 128, 9000, 1, (64, 8)),     # 8 heads: two sets of weights; many chunks, merged 8 heads at a time
    (4, 32, 128, 2500, 1, (32, 4)),
    (1, 32, 64, 2222, 1, (32, 4)),      # float32 settings
    (4, 64, 128, 2500, 3, (32, 4)),
    (4, 64, 64, 4000, 1, (32, 32)),
    (1, 32, 96, 4000, 1, (32, 8)),
])
def test_tail(bits, g, residual, n, n_new, heads):
    print(f"case tail bits={bits} g={g} W={residual} n={n} new={n_new} heads={heads}", flush=True)
    shape = HeadShape(heads[0], heads[1], 128)
    inp = make_layer(n, config=3, layer=1, seq=n % 89, shape=shape)
    layer = tkv.QuantLayer(n_q_heads=heads[0], n_kv_heads=heads[1], bits=bits, group_size=g, residual=residual,
                           capacity=(n + g) // g * g)
    kd, vd = to_new(inp.k), to_new(inp.v)
    if n > n_new:
        layer.append(kd[:, :n - n_new].contiguous(), vd[:, :n - n_new].contiguous())
    q = torch.from_numpy(inp.q)[None].cuda()
    out = layer.decode(q, SM, kd[:, n - n_new:].contiguous(), vd[:, n - n_new:].contiguous())
    ref = check_quant_cache(layer, 0, inp.k, inp.v)   # the new rows are in the ring, bit for bit
    want = attention.quant_attention(inp.q, ref, SM)
    tol = TOL_TAIL if ref.n_quant == 0 else TOL
    err = attn_err(out[0], want)
    print(f"   err {err:.3e}", flush=True)
    assert err <= tol
    again = layer.attn_decode(q, SM)                  # the same tokens, now all from the ring
    assert attn_err(again[0], want) <= tol


def float64_attention(q, k, v):
    """Eq. 3 over 4-bit keys and values in groups of 32 (residual 128), head by head on the device: Eq. 4's steps in
    float32, the rest in float64.  q [Hq, 128], k, v [n, Hkv, 128]."""
    def dequantized(x):  # [..., 32] along the last axis
        z, top = x.amin(dim=-1, keepdim=True), x.amax(dim=-1, keepdim=True)
        s = ((top.float() - z.float()) / 15.0).half()
        code = torch.where(s == 0, 0.0, ((x.float() - z.float()) / s.float()).round().clamp(0, 15))
        return code.double() * s.double() + z.double()
    n, hkv, _ = k.shape
    nq = (n - 128) // 32 * 32
    out = []
    for i in range(q.shape[0]):
        h = i // (q.shape[0] // hkv)
        if i % (q.shape[0] // hkv) == 0:
            kh, vh = k[:, h].double(), v[:, h].double()
            kh[:nq] = dequantized(k[:nq, h].view(nq // 32, 32, 128).transpose(1, 2)).transpose(1, 2).reshape(nq, 128)
            vh[:nq] = dequantized(v[:nq, h].reshape(nq, 4, 32)).reshape(nq, 128)
        out.append((vh * torch.softmax((kh * q[i].double()).sum(dim=1) * SM, dim=0)[:, None]).sum(dim=0))
    return torch.stack(out).cpu().numpy()


@pytest.mark.parametrize("heads,n,target", [
    ((64, 8), 170000, 8 * 130),   # 130 chunks x 64 heads of partials are more than the array holds, 65 are not
    ((48, 8), 220000, 8 * 170),   # groups of 6: the second workgroup has two heads
])
def test_large_groups_where_the_partials_do_not_fit(heads, n, target):
    """The entry with fixed scratch memory takes a group of 5 to 8 query heads in two workgroups (half the
    chunks) where the partials of one do not fit; many chunks come from the tuning hook here, from large
    batches of long sequences in use.  The usual split of this length is one workgroup for the group."""
    print(f"case static heads={heads} n={n} target={target}", flush=True)
    q, k, v = make_layer_device(n, n_q_heads=heads[0], n_kv_heads=heads[1], seed=5)
    layer = tkv.QuantLayer(n_q_heads=heads[0], n_kv_heads=heads[1], bits=4, group_size=32, capacity=n // 32 * 32 + 32)
    layer.append(k[None], v[None])
    want = float64_attention(q, k, v)
    assert attn_err(layer.attn_decode(q[None], SM)[0], want) <= TOL
    try:
        tkv.debug_quant_attn_config(0, target)
        got = layer.attn_decode_static(q[None], SM, torch.empty_like(q[None]))
    finally:
        tkv.debug_quant_attn_config(0, -1)
    assert attn_err(got[0], want) <= TOL


@pytest.mark.parametrize("bits,g", [(2, 32), (4, 32), (1, 64), (2, 64)])
@pytest.mark.parametrize("heads,n", [((8, 2), 800), ((16, 2), 800), ((16, 2), 2500)])
@pytest.mark.parametrize("gap", [0.0, 8.0, 16.0])
@pytest.mark.parametrize("v_old,v_recent", [(1e-3, 1e-3), (1.0, 1e-3)])
def test_blocks_keep_their_bits_beside_the_tail(bits, g, heads, n, gap, v_old, v_recent):
    """Recent tokens whose logits are `gap` nats above the rest, and small values: the quantized tokens of the waves
    that also take a piece of the tail keep a softmax reference of their own.  Bound, relative to the norm of a head's
    output: three roundings of at most 2^-11 (weight, weight times scaler, output; independent from token to token, as
    the values are, so averaging does not raise their share) and the output's spacing of 2^-24 where it is subnormal."""
    print(f"case beside the tail bits={bits} g={g} heads={heads} n={n} gap={gap} v={v_old},{v_recent}", flush=True)
    hq, hkv = heads
    inp = make_layer(n, config=2, layer=0, seq=n % 61, shape=HeadShape(hq, hkv, 128))
    k, q, v = inp.k.astype(np.float32), inp.q, inp.v.astype(np.float32) * v_old
    recent = slice(n - 129, n)
    mean = q.reshape(hkv, -1, 128).astype(np.float32).mean(axis=1)
    k[:, recent] += (gap / SM * mean / (mean ** 2).sum(axis=-1, keepdims=True))[:, None]
    v[:, recent] *= v_recent / v_old
    k, v = k.astype(np.float16), v.astype(np.float16)
    layer = tkv.QuantLayer(n_q_heads=hq, n_kv_heads=hkv, bits=bits, group_size=g, capacity=(n + g) // g * g)
    layer.append(to_new(k), to_new(v))
    want = attention.quant_attention(q, check_quant_cache(layer, 0, k, v), SM)
    out = layer.attn_decode(torch.from_numpy(q)[None].cuda(), SM)[0].float().cpu().numpy()
    norm = np.linalg.norm(want, axis=-1)
    err = np.linalg.norm(out - want, axis=-1) / norm
    print(f"   err {err.max():.3e}", flush=True)
    assert (err <= 3 * 2.0 ** -11 + 2.0 ** -25 * np.sqrt(128) / norm).all()


@pytest.mark.parametrize("bits,g", [(2, 32), (4, 32), (1, 64), (2, 64), (1, 32), (4, 64)])
@pytest.mark.parametrize("n", [300, 2500])
def test_rows_and_outputs_at_odd_addresses(bits, g, n):
    """Query, new rows and output at fp16 addresses that are no multiple of 4: sequences of one workgroup (whose threads
    write two channels each) and of several."""
    def odd(x):
        return torch.empty(x.numel() + 1, dtype=torch.float16, device="cuda")[1:].view_as(x).copy_(x)
    inp = make_layer(n, config=3, layer=1, seq=n % 89, shape=HeadShape(16, 4, 128))
    layer = tkv.QuantLayer(n_q_heads=16, n_kv_heads=4, bits=bits, group_size=g, capacity=2560)
    kd, vd = to_new(inp.k), to_new(inp.v)
    layer.append(odd(kd[:, :n - 3]), odd(vd[:, :n - 3]))
    q = torch.from_numpy(inp.q)[None].cuda()
    out = odd(torch.full_like(q, float("nan")))
    layer.decode(odd(q), SM, odd(kd[:, n - 3:]), odd(vd[:, n - 3:]), out=out)
    ref = check_quant_cache(layer, 0, inp.k, inp.v)
    assert attn_err(out[0], attention.quant_attention(inp.q, ref, SM)) <= TOL
