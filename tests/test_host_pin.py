"""CPU: the pinned host slots when their device address cannot be had.

The library runs in a child process over a few stand-ins for the HIP runtime's functions, loaded before
it: the first request for a device address fails. The slots are then not there, and the next call asks
for both again; a context that kept the host memory alone would hand kernels a null address.
"""
import os
import subprocess
import sys

STUBS = r"""
#include <stdio.h>
#include <stdlib.h>
static int asked, live;
int hipGetDeviceCount(int *n) { *n = 1; return 0; }
int hipSetDevice(int d) { return 0; }
int hipGetDevicePropertiesR0600(void *p, int d) { return 1; }
int hipGetSymbolAddress(void **p, const void *s) { *p = malloc(8); return 0; }
int hipStreamSynchronize(void *s) { return 0; }
const char *hipGetErrorString(int e) { return "stub"; }
int hipHostMalloc(void **p, size_t n, unsigned f) { *p = malloc(n); ++live; return 0; }
int hipHostFree(void *p) { free(p); --live; return 0; }
int hipHostGetDevicePointer(void **d, void *h, unsigned f) { if (asked++ == 0) return 1; *d = h; return 0; }
int stub_asked(void) { return asked; }
int stub_live(void) { return live; }
"""

CHILD = r"""
import ctypes as C, sys
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
lib = C.CDLL(sys.argv[2])
ctx = C.c_void_p()
assert lib.pb_create(C.byref(ctx), 0, None) == 0
pin = lib._ZN2pb8host_pinEP6pb_ctx
pin.argtypes = [C.c_void_p]
out = [pin(ctx), stub.stub_live(), pin(ctx), stub.stub_live(), pin(ctx), stub.stub_asked()]
lib.pb_destroy.argtypes = [C.c_void_p]
lib.pb_destroy(ctx)
print(*out, stub.stub_live())
"""


def test_no_slots_without_their_device_address(tmp_path):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    src, so = tmp_path / "stub.c", tmp_path / "stub.so"
    src.write_text(STUBS)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(so), str(src)], check=True)
    r = subprocess.run([sys.executable, "-c", CHILD, str(so), os.path.join(root, "paper_1709_08070_amd", "libpb.so")],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    # PB_EDEVICE with nothing held, then the slots, kept from then on and freed with the context
    assert [int(v) for v in r.stdout.split()] == [-3, 0, 0, 1, 0, 2, 0]
