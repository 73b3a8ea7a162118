"""The density of steps of up to 32 queries where one key has nearly all the weight: every group of keys keeps its own digits, also beside it in
a key block, for any count of (b,h)."""
import math

import pytest
import torch

import paper_2511_16047_amd as amskv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tokens", [(1, 4, 9), (1, 4, 9, 16), (1, 4, 9, 16, 25), (3, 30, 1, 7, 60, 25)])
@pytest.mark.parametrize("bh", [1, 16, 256, 257, 512, 513, 768, 1024, 1040])
@pytest.mark.parametrize("D", [64, 128])
def test_small_groups_beside_a_large_weight(D, bh, tokens):
    """The large score is about 20 in powers of two and formed in fp32: up to 8 products of 16 channels added, the scale and the exponent, rounded
    to 2^-20 each; a group's mass is added up in fewer than 2^6 steps of 2^-24.  (As the difference of two sums that hold the large weight a
    group is off by 4e-5 to 1e-3.)"""
    H = math.gcd(bh, 16)
    B, n = bh // H, len(tokens)
    args = (1, H, D, (1,) * n, tokens, B, amskv.AMSKV_DTYPE_BF16, [(0, 0, True)])
    arena = torch.empty(amskv.amskv_cache_required_bytes(*args), dtype=torch.uint8, device="cuda")
    h = amskv.amskv_cache_create(*args, arena=arena)
    g = torch.Generator(device="cuda").manual_seed(D + bh)
    mk = lambda t: torch.randn(B, H, t, D, device="cuda", generator=g).bfloat16()
    k, v, q = [mk(t) for t in tokens], [mk(t) for t in tokens], mk(tokens[-1])
    q[..., 0] = 4.0
    for x in k:
        x[..., 0] = 0.0
    k[0][..., 0, 0] = 12 * math.sqrt(D) / 4
    try:
        for s in range(n):
            amskv.amskv_append_scale(h, 0, s, k[s], v[s])
        o1, o2 = torch.empty_like(q), torch.empty_like(q)
        mass = torch.full((H, amskv.AMSKV_MAX_SCALES), float("nan"), device="cuda")
        assert amskv.amskv_attend_density(h, 0, n - 1, q, o1, mass) == list(tokens)
        amskv.amskv_attend(h, 0, n - 1, q, o2)
        torch.cuda.synchronize()
        assert torch.equal(o1.view(torch.int16), o2.view(torch.int16))
        p = torch.softmax(q.double() @ torch.cat(k, 2).double().transpose(2, 3).contiguous() / math.sqrt(D), -1)
        want = torch.stack([x.sum((2, 3)).mean(0) for x in p.split(tokens, 3)], 1)
        off = ((mass[:, :n].double() - want).abs() / want).max().item()
        assert off <= 10 * 2.0 ** -20 + 2.0 ** -18, off
    finally:
        torch.cuda.synchronize()
        amskv.amskv_cache_destroy(h)
