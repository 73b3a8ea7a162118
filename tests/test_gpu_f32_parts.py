"""fp32 attention on the bf16 matrix pipe (three parts per operand): launches large enough that the dispatch takes it, in all of its
workgroup shapes -- 8 or 4 row groups, 4 of them with the keys dealt to two -- at query counts around 32, 128 and 256, key counts that end
inside a block and a tile, and segments that end inside one fetch.  Against the oracle; cache contents bit-exact.  (The schedules of
test_forms have smaller steps too, which take the other kernel; test_f32_choice.py holds which launch takes which.)"""
import math

import pytest
import torch

import paper_2511_16047_amd as amskv
from test_gpu_parity import Runner, _qkv

pytestmark = pytest.mark.gpu

FAST = dict(layout=amskv.AMSKV_LAYOUT_PLANNED, borrow=True, fuse=True)


@pytest.mark.parametrize("flags", [{}, FAST], ids=["plain", "fast"])
@pytest.mark.parametrize("tokens", [(31, 97, 129, 64, 256, 255, 33, 160, 1), (127, 65, 225, 257, 63)])
@pytest.mark.parametrize("B,H", [(13, 8), (19, 8), (19, 16), (37, 7)])   # (the last: no multiple of the eight XCDs)
@pytest.mark.parametrize("D", [64, 128])
def test_forms(D, B, H, tokens, flags):
    sides = ((1,) * len(tokens), tokens)
    r = Runner(*sides, B, H, D, "f32", [(0, 0, True), (1, 1, False)], **flags)
    try:
        for layer in range(2):
            q, k, v = _qkv(*sides, B, H, D, "f32", 31 + layer)
            _, worst = r.run_layer(layer, q, k, v, check_cache=B == 13, units=[(0, 0), (B // 2, 1), (B - 1, H - 1)])
            # A score is off by at most 2 D / 16 + 4 roundings of a sum of D products (below 6 sqrt(D) on these inputs), times 1/sqrt(D)
            # and the slope of the exponential, and that moves O by at most the error times max |v|, which is below 6.
            assert worst <= (D / 8 + 4) * 2 ** -24 * 6 * 6
    finally:
        r.close()


def _attend(q, k, v, scale=0.0):
    B, H, t, D = q.shape
    args = (1, H, D, (1, 1), (k[0].shape[2], t), B, amskv.AMSKV_DTYPE_F32, [(0, 0, True)], scale)
    arena = torch.empty(amskv.amskv_cache_required_bytes(*args), dtype=torch.uint8, device="cuda")
    h = amskv.amskv_cache_create(*args, arena=arena)
    try:
        for s in range(2):
            amskv.amskv_append_scale(h, 0, s, k[s].contiguous(), v[s].contiguous())
        o = torch.empty_like(q)
        amskv.amskv_attend(h, 0, 1, q, o)
        torch.cuda.synchronize()
    finally:
        amskv.amskv_cache_destroy(h)
    return o


# magnitudes whose parts leave bf16's range on either side: powers of two on Q, K, V; one value that rounds to infinity in bf16; V whose
# sums do and do not overflow where they are formed
@pytest.mark.parametrize("eq,ek,ev,huge", [(0, 0, 0, False), (0, 0, 0, True), (0, 0, -118, False), (-118, 118, 0, False), (118, -118, 0, False),
                                           (-90, 90, 90, False), (0, 0, -118, True), (0, 0, 84, False), (0, 0, 94, False)])
@pytest.mark.parametrize("D,bh,tq,prev", [(64, 256, 255, 66), (64, 300, 127, 1), (64, 48, 577, 2), (128, 256, 200, 63)])
def test_magnitudes(D, bh, tq, prev, eq, ek, ev, huge):
    g = torch.Generator(device="cuda").manual_seed(tq)
    mk = lambda t, e: torch.randn(bh // 4, 4, t, D, device="cuda", generator=g) * 2.0 ** e
    q, k, v = mk(tq, eq), [mk(prev, ek), mk(tq, ek)], [mk(prev, ev), mk(tq, ev)]
    if huge:
        v[1][:, :, 7, 3] = 3.4e38
    o = _attend(q, k, v).view(bh, tq, D)
    n = prev + tq
    kk, vv = torch.cat(k, 2).view(bh, n, D), torch.cat(v, 2).view(bh, n, D)
    off, size = torch.zeros(D, dtype=torch.float64, device="cuda"), torch.zeros(D, dtype=torch.float64, device="cuda")
    for u in range(0, bh, bh // 16):
        p = torch.softmax(q.view(bh, tq, D)[u].double() @ kk[u].double().t().contiguous() / math.sqrt(D), -1) @ vv[u].double()
        off += (o[u].double() - p).pow(2).sum(0)
        size += p.pow(2).sum(0)
    rel = (off / size).sqrt().max().item()           # the worst channel: the huge value leaves the others as they are
    # a rounding is 0.43 * 2^-24 of a value in rms; n / 2 of them in a sum of n terms of either sign, about 30 in the scores (a
    # channel with one huge value has its error there alone); and a channel's figure scatters by a tenth around the whole's
    assert rel <= 1.25 * 1.25 * 0.43 * 2 ** -24 * math.sqrt(n / 2 + 30)


# Tiny values beside ordinary ones.  v: one channel; keys: every V of the keys that weigh anything; qk: a channel of K that Q makes up
# for; scale: tiny K beside a channel that Q leaves out, and a softmax scale that makes up for it
@pytest.mark.parametrize("what", ["v", "v_least", "keys", "qk", "kq", "scale"])
@pytest.mark.parametrize("D,bh,tq,prev", [(64, 256, 255, 66), (64, 300, 127, 1), (64, 48, 577, 2), (128, 256, 200, 63)])
def test_tiny_beside_ordinary(D, bh, tq, prev, what):
    g = torch.Generator(device="cuda").manual_seed(tq)
    n, scale = prev + tq, 1 / math.sqrt(D)
    q, k, v = [torch.randn(bh // 4, 4, t, D, device="cuda", generator=g) for t in (tq, n, n)]
    if what[0] == "v":
        v[..., 9] = (v[..., 9] + v[..., 9].sign()) * 2.0 ** (-116 if what == "v" else -125)  # (normal numbers)
    elif what == "keys":
        q[..., 3], k[..., 3] = 64.0, 0.0
        k[:, :, ::2, 3] = -64.0                      # scores of about -360 and less
        v[:, :, 1::2] *= 2.0 ** -116
    elif what == "scale":
        k, scale = k * 2.0 ** -116, scale * 2.0 ** 116
        q[..., 9], k[..., 9] = 0.0, 1.0
    else:
        e = 118 if what == "qk" else -118
        q[..., 9] *= 2.0 ** e
        k[..., 9] *= 2.0 ** -e
    o = _attend(q, list(k.split((prev, tq), 2)), list(v.split((prev, tq), 2)), scale).view(bh, tq, D)
    kk, vv = k.view(bh, n, D), v.view(bh, n, D)
    off, size = torch.zeros(D, dtype=torch.float64, device="cuda"), torch.zeros(D, dtype=torch.float64, device="cuda")
    for u in range(0, bh, bh // 16):
        p = torch.softmax(q.view(bh, tq, D)[u].double() @ kk[u].double().t().contiguous() * scale, -1) @ vv[u].double()
        off += (o[u].double() - p).pow(2).sum(0)
        size += p.pow(2).sum(0)
    rel = (off / size).sqrt()
    # as above; results of 2^-125 may come out in steps of 2^-149, half a step off: n of them average sqrt(n) less
    allowed = torch.full_like(rel, 1.25 * 1.25 * 0.43 * 2 ** -24 * math.sqrt(n / 2 + 30))
    if what == "v_least":
        allowed[9] += 2.0 ** -149 / (size[9] / (16 * tq)).sqrt()
    assert (rel <= allowed).all(), "%.2f of the bound" % (rel / allowed).max()


@pytest.mark.parametrize("fuse", [False, True], ids=["copied", "fused"])
@pytest.mark.parametrize("D,B,H,tq,prev", [(64, 32, 8, 255, 66), (64, 38, 8, 127, 1), (64, 6, 8, 577, 2), (128, 32, 8, 200, 63)])
def test_token_major(D, B, H, tq, prev, fuse):
    """One projection output [B][T][3][H*D] read in place, O with a padded token stride: the bits of the head-major call."""
    g = torch.Generator(device="cuda").manual_seed(tq)
    x = [torch.randn(B, t, 3, H, D, device="cuda", generator=g) for t in (prev, tq)]
    kw = dict(layout=amskv.AMSKV_LAYOUT_PLANNED, borrow_unretained=True, fuse_append=True) if fuse else {}
    args = (1, H, D, (1, 1), (prev, tq), B, amskv.AMSKV_DTYPE_F32, [(0, 0, True)])
    outs = []
    for packed in (False, True):
        arena = torch.empty(amskv.amskv_cache_required_bytes(*args, **kw), dtype=torch.uint8, device="cuda").fill_(0xFF)
        h = amskv.amskv_cache_create(*args, arena=arena, **kw)
        try:
            if packed:
                amskv.amskv_cache_set_io_layout(h, amskv.AMSKV_IO_TOKEN_MAJOR, 3 * H * D, 3 * H * D, H * D + 32)
                q, k, v = [[y[:, :, i] for y in x] for i in range(3)]
                o = [torch.zeros(B, y.shape[1], H * D + 32, device="cuda") for y in x]
            else:
                q, k, v = [[y[:, :, i].transpose(1, 2).contiguous() for y in x] for i in range(3)]
                o = [torch.zeros_like(y) for y in q]
            for s in range(2):
                amskv.amskv_append_scale(h, 0, s, k[s], v[s])
                amskv.amskv_attend(h, 0, s, q[s], o[s])
            e = torch.empty(2, B, H, prev + tq, D, device="cuda")
            amskv.amskv_cache_export(h, 0, e[0], e[1])
            torch.cuda.synchronize()
            o = o[1][:, :, : H * D].reshape(B, tq, H, D).transpose(1, 2) if packed else o[1]
            outs.append((o.contiguous().view(torch.int32), e.view(torch.int32)))
        finally:
            amskv.amskv_cache_destroy(h)
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
