"""bf16 attention of few queries on either side of the (b,h), keys and key blocks where the dispatch changes between waves of their own,
waves that share a (b,h) and workgroups of the streaming kernel, against the formula in 64 bits; and the same where the launch moves cached rows."""
import math

import numpy as np
import pytest
import torch

import paper_2511_16047_amd as amskv
from oracle import amskv_oracle as orc
from test_gpu_token_window import _segment_ids

pytestmark = pytest.mark.gpu

# queries x keys: 1 x 1, 4 x 5, 3 x 8, 1 x 9, 7 x 16, 1 x 17, 15 x 32, 32 x 64, 25 x 89, 8 x 97, 31 x 128, 33 x 161, 128 x 289, 32 x 321, 25 x 346
SIDES = ((1, 2, 1, 1, 1, 1, 3, 4, 5, 2, 1, 3, 8, 4, 5), (1, 2, 3, 1, 7, 1, 5, 8, 5, 4, 31, 11, 16, 8, 5))
TOKENS = [a * b for a, b in zip(*SIDES)]
MOST = 1040                # (b,h) from which on a wave walks alone in every launch of up to 32 queries
LINES = (1, 129, 256, 257, 384, 385, 512, 513, 768, 769, 1024, 1025)


def _run(units, D, q, k, v, each=None, **mode):
    """O of every step; each(handle, step) after it"""
    args = (1, 1, D, *SIDES, units, amskv.AMSKV_DTYPE_BF16, None if mode else [(0, 0, True)])
    arena = torch.zeros(amskv.amskv_cache_required_bytes(*args, **mode), dtype=torch.uint8, device="cuda")
    h = amskv.amskv_cache_create(*args, arena=arena, **mode)
    try:
        out = []
        for s in range(len(TOKENS)):
            a, b, c = [x[s][:units].contiguous() for x in (q, k, v)]
            o = torch.full_like(a, float("nan"))
            amskv.amskv_append_scale(h, 0, s, b, c)
            amskv.amskv_attend(h, 0, s, a, o)
            if each:
                each(h, s)
            out.append(o)
        torch.cuda.synchronize()
        return out
    finally:
        amskv.amskv_cache_destroy(h)


def _inputs(units, D, spread):
    g = torch.Generator(device="cuda").manual_seed(units + D)
    q, k, v = [[torch.randn(units, 1, n, D, generator=g, device="cuda").bfloat16() for n in TOKENS] for _ in range(3)]
    return [x * spread for x in q], k, v


def _close(o, q, k, v):
    """The kernels round each weight p and O to bf16, off by at most 2^-8 of themselves.  What the weights' errors add up to, with the weights divided by their own
    sum or by the exact one, is at most 2^-8 times the sum of p |V - O|, or of p |V|: sqrt(n) of the root of the squares' sum for n terms that count, and eight
    of its standard deviations, 8 / sqrt(3) = 4.6 of it, for many."""
    s = q.double() @ k.double().transpose(1, 2).contiguous() / math.sqrt(q.shape[-1])
    p = torch.softmax(s, -1)
    v = v.double()
    want, p2 = p @ v, p * p
    both = p2 @ (v * v), p2 @ v, p2.sum(-1, keepdim=True)
    around = (both[0] - 2 * want * both[1] + want * want * both[2]).clamp_min(0).sqrt()
    bound = 1.01 * 2.0 ** -8 * (4.6 * (around + want.abs() * both[2].sqrt()) + want.abs()) + 1e-5
    off = (o.double() - want).abs()
    assert (off <= bound).all(), (off / bound).max()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("spread", [1, 40])  # 40: a later block's scores lie far above the reference of the first
@pytest.mark.parametrize("units", LINES)
def test_every_line_of_the_dispatch(units, spread, D):
    q, k, v = _inputs(units, D, spread)
    for s, o in enumerate(_run(units, D, q, k, v)):
        _close(o[:, 0], q[s][:, 0], torch.cat(k[: s + 1], 2)[:, 0], torch.cat(v[: s + 1], 2)[:, 0])


WINDOW, SINKS = 150, 5


def _windows(units, D, spread):
    """all steps under a sliding window of tokens with sinks, and the cache bit for bit after each"""
    q, k, v = _inputs(MOST, D, spread)
    cached = orc.token_window_cache(TOKENS, WINDOW, SINKS)

    def each(h, s):
        ids = _segment_ids(TOKENS, amskv.amskv_cache_segments(h, 0))
        assert ids == cached[s]
        e = torch.empty(2, units, 1, len(ids), D, dtype=torch.bfloat16, device="cuda")
        amskv.amskv_cache_export(h, 0, e[0], e[1])
        for got, x in zip(e, (k, v)):
            assert torch.equal(got.view(torch.int16), torch.cat(x[: s + 1], 2)[:units, :, ids].view(torch.int16)), s

    return q, k, v, _run(units, D, q, k, v, each, windows=[(WINDOW, SINKS)])


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("spread", [1, 40])
@pytest.mark.parametrize("units", [1, 256, 257, 512, 513, 768, 769, 1024, MOST])
def test_moving_rows(units, spread, D):
    """wide up to 512 (b,h) (256 at head dim 128), narrow up to 1024 (768), then single waves: every (b,h) against the formula over the rows
    that the window leaves, and the cached rows as they were moved"""
    q, k, v, out = _windows(units, D, spread)
    allow, st = orc.token_window_allow_mask(TOKENS, WINDOW, SINKS), orc.scale_starts(TOKENS)
    for s, o in enumerate(out):
        ids = np.flatnonzero(allow[st[s]])
        assert (allow[st[s]: st[s] + TOKENS[s]] == allow[st[s]]).all()
        _close(o[:, 0], q[s][:units, 0], torch.cat(k, 2)[:units, 0, ids], torch.cat(v, 2)[:units, 0, ids])


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("spread", [1, 40, math.inf])
def test_workgroups_of_one_b_h_give_the_bits_of_a_single_wave(spread, D):
    """Up to 32 queries, keys not shared between waves: the same reference, sums and products in the same order, whichever kernel takes them; with
    infinite elements in every eleventh key and value as well."""
    q, k, v = _inputs(MOST, D, 1 if spread == math.inf else spread)
    if spread == math.inf:
        for x, sign in zip(k + v, [1, -1, -1] * len(k)):
            x[:, :, 3::11, 5] = sign * math.inf
    for mode in {}, {"windows": [(WINDOW, SINKS)]}:
        want = _run(MOST, D, q, k, v, **mode)
        for n in LINES:
            for s, o in enumerate(_run(n, D, q, k, v, **mode)):
                seen = sum(TOKENS[: s + 1])
                moves = mode and s == 13            # (the others with few queries have room for their rows, and share keys between waves)
                if TOKENS[s] <= 32 and (moves or seen <= 32 or n > 512):
                    same = (o.view(torch.int16) == want[s][:n].view(torch.int16)) | (o.isnan() & want[s][:n].isnan())
                    assert same.all(), (n, s, mode)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("tq,prev,units", [(9, 5, 3), (16, 14, 256), (16, 14, 513), (25, 30, 3), (25, 30, 512), (25, 30, 513), (25, 190, 513),
                                           (25, 190, 768), (32, 0, 256), (25, 190, MOST)])
def test_few_keys_are_divided_by_the_sum_of_the_rounded_weights(tq, prev, units, D):
    """Every 32nd key has the largest score and the weight 1; all others 2^-0.9945 = 0.5019, which bf16 takes to 0.5.  All V are 255/128, and so is O, where
    the rounded weights are divided by their own sum; by the sum of the unrounded ones it is 0.23 to 0.37 % smaller, and bf16's next number is 0.39 % below."""
    n, c = prev + tq, 255 / 128
    top = torch.arange(n) % 32 == 0
    k = torch.zeros(units, 1, n, D)
    k[..., ~top, 0], k[..., ~top, 1] = -1.0, 0.0055
    q = torch.zeros(units, 1, tq, D)
    q[..., :2] = 1
    q, k = q.bfloat16().cuda(), k.bfloat16().cuda()
    v = torch.full_like(k, c)
    p = torch.exp2(q[0, 0, 0].double() @ k[0, 0].double().t().contiguous())
    assert float((c * p.bfloat16().double().sum() / p.sum()).bfloat16()) < c
    sides = [x for x in (prev, tq) if x]
    args = (1, 1, D, (1,) * len(sides), sides, units, amskv.AMSKV_DTYPE_BF16, [(0, 0, True)], math.log(2.0))
    arena = torch.empty(amskv.amskv_cache_required_bytes(*args), dtype=torch.uint8, device="cuda")
    h = amskv.amskv_cache_create(*args, arena=arena)
    try:
        for s, (a, b) in enumerate(zip(k.split(sides, 2), v.split(sides, 2))):
            amskv.amskv_append_scale(h, 0, s, a.contiguous(), b.contiguous())
        o = torch.empty_like(q)
        amskv.amskv_attend(h, 0, len(sides) - 1, q, o)
        torch.cuda.synchronize()
        assert (o == c).all()
    finally:
        torch.cuda.synchronize()
        amskv.amskv_cache_destroy(h)
