"""How far attention is from the same sums in 64 bits, at the sizes of the timed cases and between them (rel: 2-norm of the
difference over 2-norm of the result, over up to 32 (b,h); printed, so that the figures quoted elsewhere can be taken again)."""
import math

import pytest
import torch

import paper_2511_16047_amd as amskv

pytestmark = pytest.mark.gpu

# (head dim, (b,h), queries, keys before them): one image to the largest batch, coarse to fine, every form of the dispatch
SHAPES = [(64, 16, 25, 30), (64, 16, 256, 424), (64, 512, 16, 14), (64, 512, 100, 155), (64, 512, 256, 424), (64, 1536, 169, 29),
          (64, 4096, 64, 105), (64, 192, 256, 0), (128, 32, 36, 21), (128, 32, 256, 165), (128, 32, 1024, 597), (128, 32, 2304, 1621),
          (128, 128, 64, 57), (128, 128, 576, 997), (128, 1024, 100, 16)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("D,bh,tq,prev", SHAPES)
def test_attention(D, bh, tq, prev, dtype):
    if dtype == "f32":
        bh = min(bh, 256)                        # (enough for the forms of fp32)
    H = math.gcd(bh, 16)
    B, n = bh // H, prev + tq
    sides = [(1, t) for t in (prev, tq) if t]
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    args = (1, H, D, *zip(*sides), B, amskv.AMSKV_DTYPE_BF16 if dtype == "bf16" else amskv.AMSKV_DTYPE_F32, [(0, 0, True)])
    arena = torch.empty(amskv.amskv_cache_required_bytes(*args), dtype=torch.uint8, device="cuda")
    h = amskv.amskv_cache_create(*args, arena=arena)
    g = torch.Generator(device="cuda").manual_seed(tq + prev)
    mk = lambda t: torch.randn(B, H, t, D, device="cuda", generator=g).to(dt)
    try:
        k, v = [mk(t) for _, t in sides], [mk(t) for _, t in sides]
        q, o = mk(tq), torch.empty(B, H, tq, D, dtype=dt, device="cuda")
        for s in range(len(sides)):
            amskv.amskv_append_scale(h, 0, s, k[s], v[s])
        amskv.amskv_attend(h, 0, len(sides) - 1, q, o)
        k, v = [torch.cat(x, 2).view(bh, n, D) for x in (k, v)]
        off = size = 0.0
        for u in range(0, bh, max(1, bh // 32)):
            p = torch.softmax(q.view(bh, tq, D)[u].double() @ k[u].double().t().contiguous() / math.sqrt(D), -1) @ v[u].double()
            off += (o.view(bh, tq, D)[u].double() - p).pow(2).sum().item()
            size += p.pow(2).sum().item()
    finally:
        torch.cuda.synchronize()
        amskv.amskv_cache_destroy(h)
    rel = math.sqrt(off / size)
    # bf16: P and O are rounded to 8 bits, 2^-9 of a value at most each.  fp32: a rounding is 0.43 * 2^-24 of a value in rms (half a
    # unit at most, uniform, over all mantissas); a sum of n terms of either sign, rounded after each, has n/2 of their squares
    # beside its own, and the scores' own roundings come to about 30 more.
    bound = math.sqrt(2) * 2 ** -9 if dtype == "bf16" else 1.25 * 0.43 * 2 ** -24 * math.sqrt(n / 2 + 30)
    print("%s, head dim %d, %d (b,h), %d x %d: rel %.3e of %.3e" % (dtype, D, bh, tq, n, rel, bound))
    assert rel <= bound
