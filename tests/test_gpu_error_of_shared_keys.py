"""bf16 attention whose key blocks are shared by several waves (slices of a unit, the two halves of a split workgroup): the error against 64
bits is that of this arithmetic, in which every share has a reference, and so a weight that is exactly 1, of its own.  One reference for all
keys is 1 to 10 % further off at these sizes."""
import math

import pytest
import torch

import paper_2511_16047_amd as amskv

pytestmark = pytest.mark.gpu

# head dim, queries, keys before them, waves that share the keys, are the weights summed as rounded?, counts of (b,h) that take this form
FORMS = [(64, 36, 55, 8, False, (16, 128)), (64, 36, 55, 2, False, (129, 256)), (64, 49, 1, 8, False, (16, 128)), (64, 49, 1, 2, False, (256,)),
         (64, 64, 91, 2, False, (256,)), (64, 100, 84, 8, False, (16, 64)), (64, 100, 84, 2, False, (128, 256)),
         (64, 16, 22, 4, True, (16, 512)), (64, 25, 30, 4, True, (16, 256, 512)), (128, 16, 22, 4, True, (16, 256)), (128, 25, 30, 4, True, (16, 256)),
         (128, 64, 91, 2, False, (16, 256)), (128, 100, 84, 2, False, (16, 128, 256))]


def _of_this_arithmetic(s, v, shares, rounded):
    """O from scores in powers of two: shares take the 32-key blocks in turn, each with the largest score of its first block as the reference"""
    blocks = s.split(32, -1)
    top = torch.stack([blocks[i].amax(-1) for i in range(min(shares, len(blocks)))], -1)
    ref = torch.cat([top[..., i % shares, None].expand_as(b) for i, b in enumerate(blocks)], -1)
    p = torch.exp2(s - ref)
    assert all(x.sum(-1).amax() <= 1024 for x in p.split(32, -1))     # (above that a reference may move)
    r = p.bfloat16().double()
    back = torch.exp2(ref - top.amax(-1, keepdim=True))
    return ((r * back) @ v / ((r if rounded else p) * back).sum(-1, keepdim=True)).bfloat16().double()


@pytest.mark.parametrize("D,tq,prev,shares,rounded,bh", [(*f[:5], n) for f in FORMS for n in f[5]])
def test_error(D, tq, prev, shares, rounded, bh):
    """rel (2-norm of the difference over 2-norm of the result) no larger than this arithmetic's.  The kernel's scores, exponentials and sums are
    fp32: off by 2^-20 at most, they take one weight in 2^11 to the other side of a rounding, 0.05 % of them; the bound has ten times that."""
    H = math.gcd(bh, 16)
    B, sides = bh // H, ((1, 1), (prev, tq))
    args = (1, H, D, *sides, B, amskv.AMSKV_DTYPE_BF16, [(0, 0, True)])
    arena = torch.empty(amskv.amskv_cache_required_bytes(*args), dtype=torch.uint8, device="cuda")
    h = amskv.amskv_cache_create(*args, arena=arena)
    g = torch.Generator(device="cuda").manual_seed(tq + prev + bh)
    mk = lambda t: torch.randn(B, H, t, D, device="cuda", generator=g).bfloat16()
    try:
        k, v = [mk(t) for t in sides[1]], [mk(t) for t in sides[1]]
        q, o = mk(tq), torch.empty(B, H, tq, D, dtype=torch.bfloat16, device="cuda")
        for s in range(2):
            amskv.amskv_append_scale(h, 0, s, k[s], v[s])
        amskv.amskv_attend(h, 0, 1, q, o)
        k, v, o = [x.flatten(0, 1).double() for x in (torch.cat(k, 2), torch.cat(v, 2), o)]
    finally:
        torch.cuda.synchronize()
        amskv.amskv_cache_destroy(h)
    s = q.flatten(0, 1).double() @ k.transpose(1, 2).contiguous() / math.sqrt(D)
    want = torch.softmax(s, -1) @ v
    rel, same, one = [((x - want).pow(2).sum() / want.pow(2).sum()).sqrt().item() for x in
                      (o, _of_this_arithmetic(s * math.log2(math.e), v, shares, rounded), _of_this_arithmetic(s * math.log2(math.e), v, 1, rounded))]
    print("head dim %d, %d (b,h), %d x %d: rel %.4e, this arithmetic %.4e, with one reference %.4e" % (D, bh, tq, tq + prev, rel, same, one))
    assert rel <= 1.005 * same


@pytest.mark.parametrize("spread", [1, 40])              # 40: references move
@pytest.mark.parametrize("D,tq,prev,wide,narrow", [(64, 33, 31, 384, 385), (64, 64, 91, 384, 385), (64, 100, 590, 384, 385), (64, 128, 1, 384, 385),
                                                   (128, 33, 31, 256, 300), (128, 36, 55, 256, 300), (128, 49, 1, 1, 300), (128, 96, 0, 256, 300)])
def test_wide_workgroups_give_the_bits_of_narrow_ones(D, tq, prev, wide, narrow, spread):
    """33 to 128 queries, keys not shared: wide up to 384 (b,h) at head dim 64, and at 128 up to 256 with up to three key blocks"""
    sides = [t for t in (prev, tq) if t]
    g = torch.Generator(device="cuda").manual_seed(tq + prev)
    mk = lambda t: torch.randn(narrow, 1, t, D, device="cuda", generator=g).bfloat16()
    k, v, q = [mk(t) for t in sides], [mk(t) for t in sides], mk(tq) * spread
    out = []
    for n in (wide, narrow):
        args = (1, 1, D, (1,) * len(sides), sides, n, amskv.AMSKV_DTYPE_BF16, [(0, 0, True)])
        arena = torch.empty(amskv.amskv_cache_required_bytes(*args), dtype=torch.uint8, device="cuda")
        h = amskv.amskv_cache_create(*args, arena=arena)
        try:
            for s in range(len(sides)):
                amskv.amskv_append_scale(h, 0, s, k[s][:n].contiguous(), v[s][:n].contiguous())
            out.append(torch.full_like(q[:n], float("nan")))
            amskv.amskv_attend(h, 0, len(sides) - 1, q[:n].contiguous(), out[-1])
        finally:
            torch.cuda.synchronize()
            amskv.amskv_cache_destroy(h)
    assert not out[1].isnan().any() and torch.equal(out[0].view(torch.int16), out[1][:wide].view(torch.int16))
