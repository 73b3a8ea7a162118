"""Eviction, compaction and append at the edges of the copying kernels: rows shorter and longer than a workgroup's
pass (128, 256 and 1024 tokens of head dim 64 in bf16; a quarter of that for 512-byte rows), rows that share a
workgroup, a last workgroup that is not full, few rows and many.  Cache contents bit-exact after every step."""
import pytest

import paper_2511_16047_amd as amskv
from test_gpu_parity import Runner, _qkv

pytestmark = pytest.mark.gpu

# 1, 12, 63, 65, 64, 192, 65, 810, 300 tokens
SIDES = ((1, 3, 7, 5, 8, 12, 13, 27, 15), (1, 4, 9, 13, 8, 16, 5, 30, 20))


@pytest.mark.parametrize("token_major", [False, True], ids=["head-major", "token-major"])
@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("f32", 128)])
@pytest.mark.parametrize("B,H", [(1, 3), (10, 13)])
def test_rolling_rows(B, H, dtype, D, token_major):
    pols = [(1, 1, False), (2, 2, False), (0, 0, True)]
    r = Runner(*SIDES, B, H, D, dtype, pols)
    try:
        if token_major:
            amskv.amskv_cache_set_io_layout(r.h, amskv.AMSKV_IO_TOKEN_MAJOR, H * D, H * D, H * D)
        for layer in range(len(pols)):
            q, k, v = _qkv(*SIDES, B, H, D, dtype, 90 + layer)
            flat = lambda x: x.permute(0, 2, 1, 3).contiguous() if token_major else x
            held = []
            for s in range(len(k)):
                held.append((flat(k[s]), flat(v[s])))
                amskv.amskv_append_scale(r.h, layer, s, *held[-1])
                r.check_cache(layer, s, k, v)
    finally:
        r.close()
