"""A call whose index lists cannot be uploaded has launched nothing when it returns: "on a non-zero return no output buffer has been
written".  On the CPU, with the HIP calls of the library answered by a small stand-in that counts launches and has no pinned memory."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2603_11243_amd", "libssd.so")

STAND_IN = r"""
#include <stdlib.h>
int launches = 0;
int hipLaunchKernel(void) { ++launches; return 0; }
int hipHostMalloc(void** p, size_t n, unsigned f) { *p = 0; return 2; }
int hipMalloc(void** p, size_t n) { *p = calloc(1, n); return 0; }
int hipFree(void* p) { free(p); return 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { *e = (void*)1; return 0; }
int hipEventDestroy(void* e) { return 0; }
int hipStreamIsCapturing(void* s, int* c) { *c = 0; return 0; }
int hipThreadExchangeStreamCaptureMode(int* m) { return 0; }
int hipMemsetAsync(void) { return 0; }
int hipMemcpyAsync(void) { return 0; }
int hipStreamSynchronize(void* s) { return 0; }
int hipFuncSetAttribute(void) { return 0; }
int hipGetLastError(void) { return 0; }
const char* hipGetErrorString(int e) { return "stand-in"; }
int __hipPushCallConfiguration(void) { return 0; }
int __hipPopCallConfiguration(void) { return 0; }
"""

CALL = r"""
import ctypes as C, sys
hip = C.CDLL(sys.argv[1], C.RTLD_GLOBAL)             # before the library: its HIP calls are bound to this
lib = C.CDLL(sys.argv[2])
lengths = [int(sys.argv[4])] + [1] * (int(sys.argv[3]) - 1)
cu = (C.c_int32 * (len(lengths) + 1))(*[sum(lengths[:b]) for b in range(len(lengths) + 1)])
p, no = C.c_void_p, C.c_void_p(None)
somewhere = p(1 << 20)                                  # device memory: the host never looks into it
h = p()
assert lib.ssd_create(C.byref(h), no, no, no) == 0
assert lib.ssd_set_ctc_head(h, somewhere, no, 348, 64) == 0
assert lib.ssd_set_workspace(h, somewhere, C.c_size_t(1 << 30)) == 0
launches = C.c_int.in_dll(hip, "launches")
out = [somewhere] * 6
for call in (lambda: lib.ctc_gate(h, somewhere, 1, cu, len(lengths), 512, 0, C.c_float(0.7), *out),
             lambda: lib.ctc_head_gate(h, somewhere, cu, len(lengths), 0, C.c_float(0.7), *out)):
    launches.value = 0
    print(call(), launches.value)
"""


# more prefix sums than arguments of a launch hold, and one length too many bits for the pairs; one utterance fewer and one frame fewer need no upload
@pytest.mark.parametrize("B,first,needs_upload", [(1281, 1, True), (300, 65536, True), (1280, 1, False), (300, 65535, False)])
def test_nothing_is_launched(tmp_path, B, first, needs_upload):
    if not os.path.exists(LIB):
        from paper_2603_11243_amd.build import build_library
        build_library(verbose=False)
    src, so = tmp_path / "stand_in.c", tmp_path / "stand_in.so"
    src.write_text(STAND_IN)
    subprocess.run(["gcc", "-w", "-shared", "-fPIC", "-o", str(so), str(src)], check=True)
    r = subprocess.run([sys.executable, "-c", CALL, str(so), LIB, str(B), str(first)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    for line in r.stdout.split("\n")[:2]:
        rc, launched = map(int, line.split())
        assert (rc, launched) == (-4, 0) if needs_upload else rc == 0 and launched >= 2, r.stdout
