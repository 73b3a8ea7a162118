"""bf16 attention of more than 32 query rows where the (b, h) are few: the dispatch chooses between workgroups of 128 and
256 rows and the form that deals a unit's key blocks to two waves.  Query and key counts around the 32-row block, the
64-key tile and the 128- and 256-row workgroups -- a last tile without, with a partial and with a whole second block --
against the oracle (max-abs 2e-2 on unit-variance inputs, as everywhere), cache contents bit-exact."""
import pytest

import amskv_inputs as inp
import paper_2511_16047_amd as amskv
from test_gpu_parity import Runner, _qkv
from test_gpu_token_window import _run as _run_window

pytestmark = pytest.mark.gpu

# 33, 64, 65, 96, 97, 128, 129, 160, 257 queries; as many keys (own scale only), with the scale before, or up to 1029
SIDES = ((3, 8, 5, 8, 1, 8, 3, 10, 1), (11, 8, 13, 12, 97, 16, 43, 16, 257))
FAST = dict(layout=amskv.AMSKV_LAYOUT_PLANNED, borrow=True, fuse=True)


@pytest.mark.parametrize("flags", [{}, FAST], ids=["plain", "fast"])
@pytest.mark.parametrize("B,H", [(1, 1), (3, 5), (9, 16), (19, 16)])   # one round of either form at most, up to several
@pytest.mark.parametrize("D", [64, 128])
def test_few_units(D, B, H, flags):
    pols = [(0, 0, False), (0, 1, False), (0, 0, True)]
    r = Runner(*SIDES, B, H, D, "bf16", pols, **flags)
    try:
        for layer in range(3):
            q, k, v = _qkv(*SIDES, B, H, D, "bf16", 71 + layer)
            every = [(b, h) for b in range(B) for h in range(H)]
            r.run_layer(layer, q, k, v, check_cache=True, units=every if len(every) <= 5 else every[:2] + every[len(every) // 2:len(every) // 2 + 2] + every[-1:])
    finally:
        r.close()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("window,n_sink", [(100, 0), (100, 1), (196, 0)])
@pytest.mark.parametrize("sides", [(10, 13, 14, 16), (5, 6, 10, 4, 12, 3)])
def test_window_over_cached_rows(sides, window, n_sink, D):
    """token window: the step's own rows land on cached rows that its queries still read"""
    _run_window(sides, 2, 3, D, "bf16", window, n_sink, inp.layer_seed(8, 300 + window), query_between=False)
