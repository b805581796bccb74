"""The record slots of the one-launch solves are used only once they have been
zeroed: after a clear that failed, the next call clears again.  Runs on the
CPU, the library on a stand-in for the few HIP calls that creating a context
and reserving its buffers make."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_2603_15910_amd import _lib

STUB = r"""
#include <stdlib.h>
#include <string.h>
static int fail_memset, fail_sync, memsets, syncs;
static size_t last_bytes;
void stand_in_fail(int memset_, int sync_) { fail_memset = memset_; fail_sync = sync_; }
int stand_in_memsets(void) { return memsets; }
size_t stand_in_bytes(void) { return last_bytes; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipSetDevice(int d) { return 0; }
int hipGetDevicePropertiesR0600(void* p, int d) { return 100; }
int hipGetSymbolAddress(void** p, const void* s) { *p = 0; return 100; }
int hipHostMalloc(void** p, size_t n, unsigned f) { *p = calloc(1, n); return 0; }
int hipHostFree(void* p) { free(p); return 0; }
int hipMalloc(void** p, size_t n) { *p = malloc(n < 1 << 22 ? n : 1 << 22); return 0; }
int hipFree(void* p) { free(p); return 0; }
int hipGetLastError(void) { return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipStreamIsCapturing(void* s, int* c) { *c = 0; return 0; }
int hipMemsetAsync(void* p, int v, size_t n, void* s) {
  ++memsets;
  last_bytes = n;
  if (fail_memset) { --fail_memset; return 1; }
  return 0;
}
int hipStreamSynchronize(void* s) {
  if (fail_sync) { --fail_sync; return 1; }
  return 0;
}
"""

PROGRAM = r"""
import ctypes as C, sys
stub = C.CDLL(sys.argv[2], mode=C.RTLD_GLOBAL)   # found before the HIP runtime
lib = C.CDLL(sys.argv[1])
stub.stand_in_bytes.restype = C.c_size_t
lib.cqk_reserve.argtypes = [C.c_void_p, C.c_int64, C.c_int32]
for fail in ((1, 0), (0, 1), (2, 0), (1, 1)):
    ctx = C.c_void_p()
    assert lib.cqk_create(C.byref(ctx), None) == 0
    stub.stand_in_fail(*fail)
    before = stub.stand_in_memsets()
    # every failed clear is followed by another one, of the same whole area
    for k in range(sum(fail) + 1):
        assert lib.cqk_reserve(ctx, 0, 0) == 0
        assert stub.stand_in_memsets() == before + k + 1, (fail, k)
        whole = stub.stand_in_bytes() if k == 0 else whole
        assert stub.stand_in_bytes() == whole > 1 << 20
    assert lib.cqk_reserve(ctx, 0, 0) == 0
    assert stub.stand_in_memsets() == before + sum(fail) + 1
    lib.cqk_destroy(ctx)
print("ok")
"""


@pytest.mark.skipif(shutil.which("gcc") is None, reason="no C compiler")
@pytest.mark.skipif(not os.path.exists(_lib.LIB_PATH), reason="the library is not built")
def test_a_failed_clear_is_repeated(tmp_path):
    src, so = tmp_path / "stand_in.c", tmp_path / "stand_in.so"
    src.write_text(STUB)
    subprocess.run(["gcc", "-w", "-shared", "-fPIC", "-o", str(so), str(src)], check=True)
    out = subprocess.run([sys.executable, "-c", PROGRAM, _lib.LIB_PATH, str(so)],
                         capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stderr
