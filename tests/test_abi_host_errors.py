"""Failures of the HIP runtime as the library's host code meets them, with no
device: the launches (and the error they leave) are a stub's, loaded ahead of
the runtime in a process of its own."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STUB = r"""
#include <stdlib.h>
static int launches, failing, last;
void stub_fail_at(int n) { failing = n; launches = 0; }
int __hipPushCallConfiguration() { return 0; }
int __hipPopCallConfiguration() { return 0; }
int stub_launches(void) { return launches; }
int hipLaunchKernel() { if (++launches != failing) return 0; return last = 719; }
int hipGetLastError(void) { int e = last; last = 0; return e; }
static int events, memory, live;
void stub_server(int e, int m) { events = e; memory = m; }
int stub_live(void) { return live; }
int hipEventCreateWithFlags(void **e) { if (events-- <= 0) return last = 100; *e = &live; ++live; return 0; }
int hipEventSynchronize() { return 0; }
int hipStreamSynchronize() { return 0; }
int hipEventDestroy() { --live; return 0; }
int hipHostMalloc(void **p, size_t n) { if (memory-- <= 0) return last = 2; *p = malloc(n); ++live; return 0; }
int hipHostGetDevicePointer(void **d, void *h) { *d = h; return 0; }
int hipHostFree(void *p) { free(p); --live; return 0; }
"""

PROGRAM = r"""
import ctypes, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
from paper_1105_5804_amd import _lib
L = _lib.lib()
W, H = 40, 30
p = _lib.SwParams(W=W, H=H, q=2, spin_kind=0, K=0.88, seed=1, stream_id=0, flags=0)
ws = L.sw_workspace_bytes(ctypes.byref(p))
base = ctypes.create_string_buffer(ws + 256)
at = ctypes.addressof(base)
at += -at % 256
spins = ctypes.create_string_buffer(W * H)
b = _lib.SwBuffers(spins=ctypes.addressof(spins), workspace=at, workspace_bytes=ws)
h = ctypes.c_void_p()
assert L.sw_init(ctypes.byref(h), ctypes.byref(p), ctypes.byref(b), None) == _lib.SW_OK
t = ctypes.c_uint64()
hist = ctypes.create_string_buffer(200 * 96)
done = 0
# 130 sweeps go out as 64 + 64 + 2: two launches, two, one
for fail_at, moved in ((1, 0), (2, 0), (3, 64), (4, 64), (5, 128), (0, 130)):
    for records in (False, True):
        stub.stub_fail_at(fail_at)
        st = (L.sw_sweep_history(h, 130, ctypes.addressof(hist), None) if records else L.sw_sweep(h, 130, None))
        assert st == (_lib.SW_OK if moved == 130 else _lib.SW_ERR_DEVICE), (fail_at, st)
        assert stub.stub_launches() == (fail_at or 5)  # nothing goes out after a launch that failed
        assert L.sw_get_t(h, ctypes.byref(t)) == _lib.SW_OK
        done += moved
        assert t.value == done, (fail_at, records, t.value, done)
assert L.sw_destroy(h) == _lib.SW_OK
print("ok")
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    d = tmp_path_factory.mktemp("stub")
    src = d / "stub.c"
    src.write_text(STUB)
    lib = d / "libstub.so"
    subprocess.check_call(["gcc", "-shared", "-fPIC", "-w", "-o", str(lib), str(src)])
    return str(lib)


def test_small_lattice_counts_the_sweeps_enqueued(stub):
    """The sweep number follows the spins when a launch fails between the
    pieces of a call."""
    r = subprocess.run([sys.executable, "-c", PROGRAM, stub, ROOT], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stderr


CREATE = r"""
import ctypes, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
from paper_1105_5804_amd import _lib
L = _lib.lib()
p = _lib.CclServerParams(_lib.CCL_SITES_OPEN, 1, 4, 1, 0)
arena = ctypes.create_string_buffer((1 << 20) + 256)
at = ctypes.addressof(arena)
at += -at % 256
h = ctypes.c_void_p()
streams = (ctypes.c_void_p * 1)(None)
for events, memory, want in ((0, 0, _lib.SW_ERR_DEVICE), (3, 1, _lib.SW_ERR_DEVICE),
                             (4, 0, _lib.SW_ERR_HOST_MEMORY), (4, 1, _lib.SW_OK)):
    stub.stub_server(events, memory)
    st = L.ccl_server_create(ctypes.byref(h), ctypes.byref(p), at, 1 << 20, streams)
    assert st == want, (events, memory, st)
    if st == _lib.SW_OK:
        assert L.ccl_server_destroy(h) == _lib.SW_OK
    assert stub.stub_live() == 0, (events, memory)  # whatever was made is given back
    assert stub.hipGetLastError() == 0  # and no error is left for another call to find
print("ok")
"""


def test_server_create_reports_what_failed(stub):
    """No device: SW_ERR_DEVICE; no pinned memory: SW_ERR_HOST_MEMORY."""
    r = subprocess.run([sys.executable, "-c", CREATE, stub, ROOT], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stderr


def test_library_of_an_older_interface_is_refused(tmp_path, monkeypatch):
    """A library built before sw_cluster_count and ccl_server_count carries a
    lower version, and the binding says that it has to be rebuilt."""
    from paper_1105_5804_amd import _lib

    src = tmp_path / "old.c"
    older = sorted(set(_lib.SIGNATURES) - {"sw_cluster_count", "ccl_server_count", "swccl_abi_version"})
    src.write_text("int swccl_abi_version(void) { return 7; }\n" + "".join(f"void {n}(void) {{}}\n" for n in older))
    lib = tmp_path / "libold.so"
    subprocess.check_call(["gcc", "-shared", "-fPIC", "-o", str(lib), str(src)])
    monkeypatch.setattr(_lib, "LIB_PATH", str(lib))
    monkeypatch.setattr(_lib, "_lib", None)
    with pytest.raises(RuntimeError, match="ABI 7.*rebuild"):
        _lib.lib()
