"""The per-layer calls take what ctypes takes: handles, addresses and streams as integers, c_void_p or whatever int() takes."""
import ctypes
import os
import subprocess
import sys
import sysconfig

import numpy as np
import pytest

import paper_2511_16047_amd as amskv
from paper_2511_16047_amd import build


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


CALLS = """
import sys
sys.modules["paper_2511_16047_amd._pycalls"] = None      # as where it is not built: importing it raises ImportError
import paper_2511_16047_amd as amskv
from paper_2511_16047_amd import build
h = amskv.amskv_cache_create(1, 2, 64, (1, 2), (1, 2), 1, amskv.AMSKV_DTYPE_BF16, [(1, 1, False)])
amskv.amskv_append_scale(h, 0, 0)
for call in (lambda: amskv.amskv_append_scale(h, 0, 0, None, None, 0), lambda: amskv.amskv_attend(h, 0, 0, 4096, 8192)):
    try:
        call()
    except amskv.AmskvError as e:
        print(e.status)
amskv.amskv_cache_destroy(h)
"""


def test_without_the_extension_module_the_calls_go_through_ctypes():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    p = subprocess.run([sys.executable, "-c", CALLS], cwd=root, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, p.stdout
    assert p.stdout.split() == [str(amskv.AMSKV_ERR_ORDER), str(amskv.AMSKV_ERR_NO_DEVICE_MEMORY)]


def test_the_extension_module_is_named_for_its_interpreter():
    assert os.path.basename(build.PYCALLS) == "_pycalls" + sysconfig.get_config_var("EXT_SUFFIX")
    assert os.path.exists(build.PYCALLS)


def test_a_torch_without_the_raw_stream_functions_is_asked_the_public_way(monkeypatch):
    import types
    import torch
    from paper_2511_16047_amd import binding
    for name in ("_cuda_getDevice", "_cuda_getCurrentRawStream"):
        monkeypatch.delattr(torch._C, name, raising=False)
    monkeypatch.setattr(torch.cuda, "is_available", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda d=None: types.SimpleNamespace(cuda_stream=0 if d is None else 100 + d))
    monkeypatch.setattr(binding, "_lookup", None)
    assert binding._stream(None) == 103
