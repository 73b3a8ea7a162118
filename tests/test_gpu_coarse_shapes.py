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
    # bf16 has 8 bits: a weight is off by 2^-8 of itself at most, which moves the mean of the V by 2^-8 of the farthest one's distance from it
    # (|V| is below 6 here), and so is O.  (2^-9 was assumed for both at first: half of what the rounding may be, and exceeded in earnest
    # by steps of more than 32 queries, whose kernels have not changed: 1.66 times 2^-9 * (5 + |O|).)
    assert ((o.double() - want).abs() <= 2.0 ** -8 * (6.0 + 2.0 * want.abs())).all(), (o.double() - want).abs().max()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("spread", [1, 40])  # 40: a later block's scores lie far above the reference of the first
@pytest.mark.parametrize("units", [1, 129, 256, 257, 384, 385, 512, 513, 768, 769, 1024, 1025])
def test_every_line_of_the_dispatch(units, spread, D):
    q, k, v = _inputs(units, 1, D)
    q = [x * spread for x in q]
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


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("units", [3, 256, 513])
def test_few_keys_are_divided_by_the_sum_of_the_rounded_weights(units, D):
    """O times the sum that the weights are divided by is a sum of the rounded weights: with all V equal to one number, O is that number,
    bit for bit (its own rounding of 2^-24 and the quotient's do not reach bf16's last bit)."""
    q, k, v = _inputs(units, 1, D)
    v = [torch.full_like(x, 1.5) for x in v]
    out, _ = _run(units, 1, D, q, k, v)
    for s, o in enumerate(out):
        if o.shape[2] <= 32 and sum(x.shape[2] for x in k[: s + 1]) <= 97:
            assert (o == 1.5).all()
