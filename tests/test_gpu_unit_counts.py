"""The attention kernels' dispatch depends on how many (b, h, query block) units a step has and on how many keys they
walk: every variant at its edges -- query counts around a tile, key counts around a block, one unit up to more than
fill the chip -- against the oracle (max-abs 1e-4 fp32, 2e-2 bf16 on unit-variance inputs, as everywhere), cache
contents bit-exact."""
import pytest

import paper_2511_16047_amd as amskv
from test_gpu_parity import Runner, _qkv

pytestmark = pytest.mark.gpu

# 1, 16, 17, 31, 33, 64, 130 queries; 1 to 292 keys
SIDES = ((1, 4, 1, 31, 3, 8, 10), (1, 4, 17, 1, 11, 8, 13))
FAST = dict(layout=amskv.AMSKV_LAYOUT_PLANNED, borrow=True, fuse=True)


def _units(B, H):
    every = [(b, h) for b in range(B) for h in range(H)]
    return every if len(every) <= 12 else every[:3] + every[len(every) // 2: len(every) // 2 + 5] + every[-4:]


@pytest.mark.parametrize("flags", [{}, FAST], ids=["plain", "fast"])
@pytest.mark.parametrize("B,H", [(1, 1), (3, 5), (5, 8), (13, 20), (35, 32)])
@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128)])
def test_every_unit_count(dtype, D, B, H, flags):
    pols = [(0, 0, True), (1, 1, False)]
    r = Runner(*SIDES, B, H, D, dtype, pols, **flags)
    try:
        for layer in range(2):
            q, k, v = _qkv(*SIDES, B, H, D, dtype, 41 + layer)
            r.run_layer(layer, q, k, v, check_cache=B * H <= 40, units=_units(B, H))
    finally:
        r.close()
