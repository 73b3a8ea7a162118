"""bf16 attention of few queries on either side of the (b,h), keys and key blocks where the dispatch changes between waves of their own and
workgroups of the streaming kernel, against the formula in 64 bits; and the same where the launch moves cached rows."""
import pytest
import torch

import paper_2511_16047_amd as amskv

pytestmark = pytest.mark.gpu

# queries x keys: 1 x 1, 4 x 5, 3 x 8, 1 x 9, 7 x 16, 1 x 17, 15 x 32, 32 x 64, 25 x 89, 8 x 97, 31 x 128, 33 x 161, 128 x 289, 32 x 321, 25 x 346
SIDES = ((1, 2, 1, 1, 1, 1, 3, 4, 5, 2, 1, 3, 8, 4, 5), (1, 2, 3, 1, 7, 1, 5, 8, 5, 4, 31, 11, 16, 8, 5))


def _run(B, H, D, q, k, v, **mode):
    """O of every step and the cached K, V at the end."""
    args = (1, H, D, *SIDES, B, amskv.AMSKV_DTYPE_BF16, None if mode else [(0, 0, True)])
    arena = torch.zeros(amskv.amskv_cache_required_bytes(*args, **mode), dtype=torch.uint8, device="cuda")
    h = amskv.amskv_cache_create(*args, arena=arena, **mode)
    try:
        out = []
        for s in range(len(q)):
            o = torch.full_like(q[s], float("nan"))
            amskv.amskv_append_scale(h, 0, s, k[s], v[s])
            amskv.amskv_attend(h, 0, s, q[s], o)
            out.append(o)
        torch.cuda.synchronize()
        return out, arena
    finally:
        amskv.amskv_cache_destroy(h)


def _inputs(B, H, D):
    g = torch.Generator(device="cuda").manual_seed(B * H + D)
    t = [a * b for a, b in zip(*SIDES)]
    return [[torch.randn(B, H, n, D, generator=g, device="cuda").bfloat16() for n in t] for _ in range(3)]


def _close(o, want):
    # P and O are rounded to bf16: 2^-9 of the largest |V| (below 5 here) each, and 2^-9 of O itself
    assert ((o.double() - want).abs() <= 2.0 ** -9 * (5.0 + want.abs())).all(), (o.double() - want).abs().max()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("units", [1, 129, 256, 257, 384, 385, 512, 513, 768, 769, 1024, 1025])
def test_every_line_of_the_dispatch(units, D):
    q, k, v = _inputs(units, 1, D)
    out, _ = _run(units, 1, D, q, k, v)
    for s, o in enumerate(out):
        ks, vs = (torch.cat(x[: s + 1], 2)[:, 0].double() for x in (k, v))
        p = torch.softmax(q[s][:, 0].double() @ ks.transpose(1, 2).contiguous() / D ** 0.5, -1)
        _close(o[:, 0], p @ vs)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("units", [257, 513, 769, 1025])
def test_moving_rows(units, D):
    """a sliding window of tokens with sinks: all (b,h) in one cache, and the first three in one of their own, which takes the form that is
    checked against the oracle elsewhere"""
    q, k, v = _inputs(units, 1, D)
    mode = {"windows": [(150, 5)]}
    out, _ = _run(units, 1, D, q, k, v, **mode)
    few, _ = _run(3, 1, D, *[[x[:3].contiguous() for x in t] for t in (q, k, v)], **mode)
    for o, want in zip(out, few):
        _close(o[:3], want.double())
