"""The per-layer calls take what ctypes takes: handles, addresses and streams as integers, c_void_p or whatever int() takes."""
import ctypes

import numpy as np
import pytest

import paper_2511_16047_amd as amskv


@pytest.mark.parametrize("handle", [int, ctypes.c_void_p], ids=["int", "c_void_p"])
@pytest.mark.parametrize("stream", [None, 0, np.uint64(0), ctypes.c_void_p(0).value], ids=["none", "zero", "numpy", "null"])
def test_forms_of_handle_and_stream(handle, stream):
    h = amskv.amskv_cache_create(1, 2, 64, (1, 2, 3), (1, 2, 3), 1, amskv.AMSKV_DTYPE_BF16, [(1, 1, False)])
    try:
        for s in range(3):
            amskv.amskv_append_scale(handle(h), 0, s, None, None, stream)     # plan only: no device memory
        with pytest.raises(amskv.AmskvError) as e:
            amskv.amskv_append_scale(handle(h), 0, 0, None, None, stream)
        assert e.value.status == amskv.AMSKV_ERR_ORDER
        with pytest.raises(amskv.AmskvError) as e:
            amskv.amskv_attend(handle(h), 0, 2, 4096, 8192, stream)
        assert e.value.status == amskv.AMSKV_ERR_NO_DEVICE_MEMORY
    finally:
        amskv.amskv_cache_destroy(h)


def test_a_wrong_argument_is_still_refused():
    with pytest.raises((TypeError, ctypes.ArgumentError)):
        amskv.amskv_append_scale(object(), 0, 0)
