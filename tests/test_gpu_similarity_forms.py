"""Inter-scale similarity: both workgroup sizes at every dtype and head dim, on either side of where the dispatch changes
between them (512 and 256 (b,h), 32 and 16 KB of a (b,h)'s rows), with less than a pass, ragged passes and many of them."""
import numpy as np
import pytest
import torch

import paper_2511_16047_amd as amskv
from oracle import amskv_oracle as orc

pytestmark = pytest.mark.gpu

# 1, 6, 35, 64, 143, 256, 270 tokens, up to 540 in the narrow ones
SIDES = ((1, 2, 5, 8, 11, 16, 10, 20), (1, 3, 7, 8, 13, 16, 27, 27))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,H", [(1, 2), (15, 17), (17, 16), (73, 7), (32, 16)])      # 2, 255, 272, 511, 512
def test_both_forms(B, H, dtype, D):
    """the cosine to 1e-5 of the oracle; the keys' sums bit for bit the same with and without the values"""
    sides = list(zip(*SIDES))
    dt = amskv.AMSKV_DTYPE_BF16 if dtype == "bf16" else amskv.AMSKV_DTYPE_F32
    args = (1, H, D, *SIDES, B, dt, [(0, 0, True)])
    arena = torch.empty(amskv.amskv_cache_required_bytes(*args), dtype=torch.uint8, device="cuda")
    h = amskv.amskv_cache_create(*args, arena=arena)
    g = torch.Generator().manual_seed(B + D)
    last = None
    try:
        for s, (a, b) in enumerate(sides):
            k, v = torch.randn(2, B, H, a * b, D, generator=g)
            if s:
                k = 0.6 * k + 0.8 * torch.from_numpy(orc.bilinear_upsample(last.double().numpy(), *sides[s - 1], a, b)).float()
            k, v = [x.to(torch.bfloat16 if dtype == "bf16" else torch.float32) for x in (k, v)]
            amskv.amskv_append_scale(h, 0, s, k.cuda(), v.cuda())
            torch.cuda.synchronize()
            if s:
                alone, both = torch.zeros(H * 4, device="cuda"), torch.zeros(2 * H * 4, device="cuda")
                amskv.amskv_interscale_similarity_enqueue_static(h, 0, s, False, alone)
                amskv.amskv_interscale_similarity_enqueue_static(h, 0, s, True, both)
                assert torch.equal(alone, both[: H * 4])
                want, _ = orc.interscale_similarity(k.double().numpy(), last.double().numpy(), (a, b), sides[s - 1])
                np.testing.assert_allclose(alone.view(H, 4)[:, 0].double().cpu().numpy() / (B * a * b), want, rtol=0, atol=1e-5)
            last = k
    finally:
        amskv.amskv_cache_destroy(h)
