"""The span of a timed call holds all of its launches.  On the CPU, with the HIP calls of the library answered by a stand-in that notes
how many launches lie before every event."""
import os
import subprocess
import sys

import pytest

from tests.test_failed_upload import LIB, STAND_IN

NOTES = r"""
int marks[16], n_marks = 0;
int hipEventCreate(void** e) { *e = (void*)1; return 0; }
int hipEventRecord(void* e, void* s) { if (n_marks < 16) marks[n_marks++] = launches; return 0; }
"""

CALL = r"""
import ctypes as C, sys
hip = C.CDLL(sys.argv[1], C.RTLD_GLOBAL)             # before the library: its HIP calls are bound to this
lib = C.CDLL(sys.argv[2])
B, frames = int(sys.argv[3]), int(sys.argv[4])
cu = (C.c_int32 * (B + 1))(*[frames * b for b in range(B + 1)])
p, no = C.c_void_p, C.c_void_p(None)
somewhere = p(1 << 20)                                  # device memory: the host never looks into it
h = p()
assert lib.ssd_create(C.byref(h), no, no, no) == 0
assert lib.ssd_set_qformer(h, somewhere, somewhere, somewhere, somewhere, 3, 16, 1024, 1024, 256, 15) == 0
assert lib.ssd_set_workspace(h, somewhere, C.c_size_t(1 << 40)) == 0
assert lib.ssd_profile_select(h, -1) == 0
before = C.c_int.in_dll(hip, "launches").value
C.c_int.in_dll(hip, "n_marks").value = 0
assert lib.qformer_pool(h, somewhere, cu, B, somewhere, (C.c_int32 * (B + 1))()) == 0
n = C.c_int.in_dll(hip, "n_marks").value
print(*[m - before for m in (C.c_int * 16).in_dll(hip, "marks")[:n]], C.c_int.in_dll(hip, "launches").value - before)
"""


# the windows as arguments; listed on the device, values projected before and after the pooling
@pytest.mark.parametrize("B,frames", [(2, 100), (500, 20), (500, 60)])
def test_projector_span(tmp_path, B, frames):
    if not os.path.exists(LIB):
        from paper_2603_11243_amd.build import build_library
        build_library(verbose=False)
    src, so = tmp_path / "stand_in.c", tmp_path / "stand_in.so"
    src.write_text(STAND_IN + NOTES)
    subprocess.run(["gcc", "-w", "-shared", "-fPIC", "-o", str(so), str(src)], check=True)
    r = subprocess.run([sys.executable, "-c", CALL, str(so), LIB, str(B), str(frames)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    begin, end, launched = map(int, r.stdout.split())
    assert begin == 0 and end == launched >= 3
