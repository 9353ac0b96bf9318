"""Argument errors of the calls that hand counts to the host (no device work)."""
import ctypes

from paper_1105_5804_amd import _lib


def test_count_argument_errors():
    L = _lib.lib()
    n64, n32 = ctypes.c_int64(), ctypes.c_int32()
    assert L.sw_cluster_count(None, ctypes.byref(n64), None) == _lib.SW_ERR_ARG
    assert L.ccl_server_count(None, 0, ctypes.byref(n32)) == _lib.SW_ERR_ARG
