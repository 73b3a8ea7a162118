"""amskv_attend_density on every form of the bf16 attention: waves of a workgroup sharing a unit, split, narrow and wide
workgroups, and the launches that move cached rows while their queries read them (token modes, up to 256 queries at head dim 64).
O and the cache bit for bit as amskv_attend leaves them on a twin cache; the masses to 2e-4 (1e-5 absolute) of 64 bits, as
everywhere (fp32 sums of exponentials of exact bf16 products)."""
import numpy as np
import pytest
import torch

import amskv_inputs as inp
import paper_2511_16047_amd as amskv
from oracle import amskv_oracle as orc
from test_gpu_density import _bits, _f64, _mass_rows, _runs_by_scale
from test_gpu_token_window import _segment_ids

pytestmark = pytest.mark.gpu

BF16 = amskv.AMSKV_DTYPE_BF16


def _twins(layers, H, D, sh, sw, B, pols, **kw):
    args = (layers, H, D, sh, sw, B, BF16, pols)
    arenas = [torch.empty(amskv.amskv_cache_required_bytes(*args, **kw), dtype=torch.uint8, device="cuda").fill_(0xFF) for _ in range(2)]
    return arenas, [amskv.amskv_cache_create(*args, arena=a, **kw) for a in arenas]


# 1, 6, 36, 64, 100, 128, 129, 270 tokens: groups that end inside a block, at its end, and in a block of the other slice
SIDES = ((1, 2, 6, 8, 10, 8, 3, 10), (1, 3, 6, 8, 10, 16, 43, 27))
FAST = dict(layout=amskv.AMSKV_LAYOUT_PLANNED, borrow_unretained=True, fuse_append=True)


@pytest.mark.parametrize("flags", [{}, FAST], ids=["plain", "fast"])
@pytest.mark.parametrize("B,H", [(1, 3), (9, 16), (20, 16)])
@pytest.mark.parametrize("D", [64, 128])
def test_scale_windows(D, B, H, flags):
    pols = [(0, 0, True), (1, 1, False)]
    tokens = [a * b for a, b in zip(*SIDES)]
    _, (one, two) = _twins(len(pols), H, D, *SIDES, B, pols, **flags)
    g = torch.Generator(device="cuda").manual_seed(D + B)
    mk = lambda t: torch.randn(B, H, t, D, device="cuda", generator=g).bfloat16()
    k_all = []
    try:
        for s, t in enumerate(tokens):
            q, k, v = mk(t), mk(t), mk(t)
            k_all.append(k)
            for l, pol in enumerate(pols):
                for h in (one, two):
                    amskv.amskv_append_scale(h, l, s, k, v)
                o1, o2 = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
                mass = torch.full((H, amskv.AMSKV_MAX_SCALES), float("nan"), device="cuda")
                lens = amskv.amskv_attend_density(one, l, s, q, o1, mass)
                amskv.amskv_attend(two, l, s, q, o2)
                torch.cuda.synchronize()
                kept = orc.kept_scales(pol, s)
                assert lens == [tokens[j] for j in kept]
                assert torch.equal(o1.view(torch.int16), o2.view(torch.int16)), (s, l)
                p = torch.softmax(q.double() @ torch.cat([k_all[j] for j in kept], 2).double().transpose(2, 3).contiguous() / D ** 0.5, -1)
                want = torch.stack([x.sum((2, 3)).mean(0) for x in p.split(lens, 3)], 1)
                got = mass[:, : len(lens)].double()
                assert torch.allclose(got, want, rtol=2e-4, atol=1e-5), (s, l, (got - want).abs().max())
        for l, pol in enumerate(pols):
            tk = sum(tokens[j] for j in orc.kept_scales(pol, len(tokens) - 1))
            e = torch.empty(4, B, H, tk, D, dtype=torch.bfloat16, device="cuda")
            amskv.amskv_cache_export(one, l, e[0], e[1])
            amskv.amskv_cache_export(two, l, e[2], e[3])
            torch.cuda.synchronize()
            assert torch.equal(e[:2].view(torch.int16), e[2:].view(torch.int16))
    finally:
        amskv.amskv_cache_destroy(one)
        amskv.amskv_cache_destroy(two)


# 144, 196, 256 and 169, 121 queries: one eight-wave workgroup moves the rows of a (b,h) at head dim 64; up to 128 (100, 64)
# the split form does; the windows cut the newest scale, land it on cached rows, keep sinks or not
@pytest.mark.parametrize("sides", [(12, 14, 16, 13, 10), (3, 8, 11, 16, 15, 4)])
@pytest.mark.parametrize("window,n_sink", [(100, 0), (150, 6), (196, 0), (300, 5)])
@pytest.mark.parametrize("D,B,H", [(64, 2, 3), (128, 1, 2), (64, 20, 16)])
def test_token_windows_move_rows(D, B, H, window, n_sink, sides):
    tokens = [x * x for x in sides]
    st = orc.scale_starts(tokens)
    if B * H <= 6:
        q, k, v = inp.correlated_qkv(sides, B, H, D, "bf16", inp.layer_seed(8, 800 + window), 0.6)
    else:                                       # a few units, repeated: every copy must come out the same
        q, k, v = ([x.repeat(B // 2, H // 2, 1, 1) for x in t] for t in inp.correlated_qkv(sides, 2, 2, D, "bf16", 5 + window, 0.6))
    small = [[x[:2, :6] for x in t] for t in (q, k, v)] if B * H <= 6 else [[x[:2, :2] for x in t] for t in (q, k, v)]
    qs, ks, vs = (np.concatenate([_f64(x) for x in t], axis=-2) for t in small)
    allow = orc.token_window_allow_mask(tokens, window, n_sink)
    cached = orc.token_window_cache(tokens, window, n_sink)
    want_o = orc.masked_attention(qs, ks, vs, allow)
    qd, kd, vd = ([x.cuda().contiguous() for x in t] for t in (q, k, v))
    arenas, (one, two) = _twins(1, H, D, sides, sides, B, None, windows=[(window, n_sink)])
    try:
        for s in range(len(sides)):
            for h in (one, two):
                amskv.amskv_append_scale(h, 0, s, kd[s], vd[s])
            o1, o2 = torch.full_like(qd[s], float("nan")), torch.full_like(qd[s], float("nan"))
            mass = torch.full((H * amskv.AMSKV_MAX_SCALES,), float("nan"), device="cuda")
            lens = amskv.amskv_attend_density(one, 0, s, qd[s], o1, mass)
            amskv.amskv_attend(two, 0, s, qd[s], o2)
            torch.cuda.synchronize()
            assert np.array_equal(_bits(o1), _bits(o2)), s
            assert np.abs(_f64(o1[: len(qs), : qs.shape[1]]) - want_o[..., st[s]: st[s] + tokens[s], :]).max() <= 2e-2
            pieces = _runs_by_scale((cached[s - 1] if s else []) + list(range(st[s], st[s] + tokens[s])), tokens)
            assert lens == [n for _, n in pieces]
            _, want_m = orc.attention_density(_f64(small[0][s]), ks, allow[st[s]: st[s] + tokens[s]], pieces)
            got_m = _mass_rows(mass, H, len(lens))[: len(want_m)]
            assert np.allclose(got_m, want_m, rtol=2e-4, atol=1e-5), (s, np.abs(got_m - want_m).max())
            for h in (one, two):
                ids = _segment_ids(tokens, amskv.amskv_cache_segments(h, 0))
                assert ids == cached[s]
                e = torch.empty(2, B, H, max(1, len(ids)), D, dtype=torch.bfloat16, device="cuda")
                if ids:
                    amskv.amskv_cache_export(h, 0, e[0], e[1])
                    torch.cuda.synchronize()
                    assert np.array_equal(_bits(e[0]), np.concatenate([_bits(x) for x in kd], axis=-2)[..., ids, :])
                    assert np.array_equal(_bits(e[1]), np.concatenate([_bits(x) for x in vd], axis=-2)[..., ids, :])
    finally:
        amskv.amskv_cache_destroy(one)
        amskv.amskv_cache_destroy(two)


@pytest.mark.parametrize("theta", [-2.0, 2.0], ids=["holds", "grows"])
@pytest.mark.parametrize("D", [64, 128])
def test_token_budget_decided_on_the_device(D, theta):
    """the launch is handed both outcomes of the Eq. 3 test and moves the rows of the one that came out"""
    sides, B, H = (10, 11, 13, 16, 12), 2, 3
    tokens = [x * x for x in sides]
    st = orc.scale_starts(tokens)
    q, k, v = inp.correlated_qkv(sides, B, H, D, "bf16", inp.layer_seed(8, 900 + D), 0.6)
    qd, kd, vd = ([x.cuda() for x in t] for t in (q, k, v))
    budget = (260, 330, 7, theta)
    trace = orc.alg1_cache_trace(tokens, *budget[:3], [theta > 1.0] * len(sides))
    ks = np.concatenate([_f64(x) for x in k], axis=-2)
    allow = orc.alg1_allow_mask(tokens, trace)
    arenas, (one, two) = _twins(1, H, D, sides, sides, B, None, budgets=[budget])
    try:
        for s in range(len(sides)):
            for h in (one, two):
                amskv.amskv_append_scale(h, 0, s, kd[s], vd[s])
            o1, o2 = torch.full_like(qd[s], float("nan")), torch.full_like(qd[s], float("nan"))
            mass = torch.full((H * amskv.AMSKV_MAX_SCALES,), float("nan"), device="cuda")
            lens = amskv.amskv_attend_density(one, 0, s, qd[s], o1, mass)
            amskv.amskv_attend(two, 0, s, qd[s], o2)
            torch.cuda.synchronize()
            assert np.array_equal(_bits(o1), _bits(o2)), s
            pieces = _runs_by_scale((trace[s - 1][0] if s else []) + list(range(st[s], st[s] + tokens[s])), tokens)
            assert lens == [n for _, n in pieces]
            _, want_m = orc.attention_density(_f64(q[s]), ks, allow[st[s]: st[s] + tokens[s]], pieces)
            assert np.allclose(_mass_rows(mass, H, len(lens)), want_m, rtol=2e-4, atol=1e-5), s
            for h in (one, two):
                ids = _segment_ids(tokens, amskv.amskv_cache_segments(h, 0))
                assert ids == trace[s][0] and amskv.amskv_cache_budget_tokens(h, 0) == trace[s][1]
                e = torch.empty(2, B, H, len(ids), D, dtype=torch.bfloat16, device="cuda")
                amskv.amskv_cache_export(h, 0, e[0], e[1])
                torch.cuda.synchronize()
                assert np.array_equal(_bits(e[0]), np.concatenate([_bits(x) for x in k], axis=-2)[..., ids, :])
                assert np.array_equal(_bits(e[1]), np.concatenate([_bits(x) for x in v], axis=-2)[..., ids, :])
    finally:
        amskv.amskv_cache_destroy(one)
        amskv.amskv_cache_destroy(two)


# keys that grow from scale to scale, so that the softmax reference moves in blocks that groups end in: wide, narrow, split
@pytest.mark.parametrize("bh,tq", [(256, 250), (512, 100), (128, 97)])
@pytest.mark.parametrize("D", [64, 128])
def test_moving_references(D, bh, tq):
    H, tokens = 8, (1, 6, 36, 64, 200, tq)
    B, pols = bh // H, [(0, 0, True)]
    _, (one, two) = _twins(1, H, D, (1,) * 6, tokens, B, pols, **FAST)
    g = torch.Generator(device="cuda").manual_seed(bh)
    mk = lambda t, a: (torch.randn(B, H, t, D, device="cuda", generator=g) * a).bfloat16()
    k = [mk(t, 1 + 1.2 * s) for s, t in enumerate(tokens)]
    v, q = [mk(t, 1) for t in tokens], [mk(t, 1) for t in tokens]
    mass = torch.full((H, amskv.AMSKV_MAX_SCALES), float("nan"), device="cuda")
    try:
        for s in range(6):
            for h in (one, two):
                amskv.amskv_append_scale(h, 0, s, k[s], v[s])
            o1, o2 = torch.full_like(q[s], float("nan")), torch.full_like(q[s], float("nan"))
            lens = amskv.amskv_attend_density(one, 0, s, q[s], o1, mass)
            amskv.amskv_attend(two, 0, s, q[s], o2)
            torch.cuda.synchronize()
            assert torch.equal(o1.view(torch.int16), o2.view(torch.int16)), s
            p = torch.softmax(q[s].double() @ torch.cat(k[: s + 1], 2).double().transpose(2, 3).contiguous() / D ** 0.5, -1)
            want = torch.stack([x.sum((2, 3)).mean(0) for x in p.split(lens, 3)], 1)
            assert torch.allclose(mass[:, : len(lens)].double(), want, rtol=2e-4, atol=1e-5), s
    finally:
        amskv.amskv_cache_destroy(one)
        amskv.amskv_cache_destroy(two)
