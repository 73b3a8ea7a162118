"""Inter-scale similarity: the form with a wave per (b,h), on either side of where the dispatch changes to it (4 KB of a (b,h)'s rows, four
bytes of them per (b,h)), with a last workgroup that is not full and with less than a pass, ragged passes and up to four of them."""
import numpy as np
import pytest
import torch

import paper_2511_16047_amd as amskv
from oracle import amskv_oracle as orc

pytestmark = pytest.mark.gpu

# 1, 2, 6, 8, 9, 15, 16, 17, 31, 32, 33 tokens
SIDES = ((1, 1, 2, 2, 3, 3, 4, 1, 1, 4, 3), (1, 2, 3, 4, 3, 5, 4, 17, 31, 8, 11))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,H", [(3, 11), (37, 7), (511, 1), (73, 14), (65, 17)])      # 33, 259, 511, 1022, 1105
def test_wave_form(B, H, dtype, D):
    """All four sums of either tensor against the oracle's 64 bits.  Each is a sum of B * T terms, formed over at most 4 passes, 64 lanes and B / 64 + 6
    steps of the batch from dot products of at most 128 channels: fewer than 64 roundings of fp32 in a row, 64 * 2^-24 = 4e-6 of the
    sum of the terms' sizes."""
    sides = list(zip(*SIDES))
    dt = amskv.AMSKV_DTYPE_BF16 if dtype == "bf16" else amskv.AMSKV_DTYPE_F32
    args = (1, H, D, *SIDES, B, dt, [(0, 0, True)])
    arena = torch.empty(amskv.amskv_cache_required_bytes(*args), dtype=torch.uint8, device="cuda")
    h = amskv.amskv_cache_create(*args, arena=arena)
    g = torch.Generator().manual_seed(B + D)
    last = None
    try:
        for s, (a, b) in enumerate(sides):
            kv = torch.randn(2, B, H, a * b, D, generator=g)
            if s:
                kv = 0.6 * kv + 0.8 * torch.from_numpy(orc.bilinear_upsample(last.double().numpy(), *sides[s - 1], a, b)).float()
            kv = kv.to(torch.bfloat16 if dtype == "bf16" else torch.float32)
            amskv.amskv_append_scale(h, 0, s, kv[0].cuda(), kv[1].cuda())
            if s:
                alone, both = torch.zeros(H * 4, device="cuda"), torch.full((2, H, 4), float("nan"), device="cuda")
                amskv.amskv_interscale_similarity_enqueue_static(h, 0, s, False, alone)
                amskv.amskv_interscale_similarity_enqueue_static(h, 0, s, True, both)
                assert torch.equal(alone.view(H, 4), both[0])
                up = torch.from_numpy(orc.bilinear_upsample(last.double().numpy(), *sides[s - 1], a, b))
                x = kv.double()
                ab, aa, bb = (x * up).sum(-1), (x * x).sum(-1), (up * up).sum(-1)
                for i, (term, size) in enumerate(((ab / (aa * bb).sqrt(), None), (ab, (x * up).abs().sum(-1)), (aa, None), (bb, None))):
                    want, scale = term.sum((1, 3)), (term.abs() if size is None else size).sum((1, 3))
                    # (the cosine is a quotient: its numerator's error counts relative to |a||b|, not to itself)
                    scale = torch.full_like(scale, float(B * a * b)) if i == 0 else scale
                    got = both[:, :, i].double().cpu()
                    assert ((got - want).abs() <= 4e-6 * scale).all(), (s, i, ((got - want).abs() / scale).max())
            last = kv
    finally:
        amskv.amskv_cache_destroy(h)
