"""The launch paths of the C ABI on a stand-in for the HIP runtime (no GPU): what they report when a launch cannot be made.

The stand-in is loaded before the library and takes the place of the runtime's functions: device memory is host memory, launches
are counted and not run, and the number of compute units is whatever the test says."""
import json
import os
import subprocess
import sys

import pytest

from paper_2504_20490_amd import build as lib_build

STAND_IN = r"""
#include <stdlib.h>
#include <string.h>
static int launches, units = 256;
int fake_launches(void) { return launches; }
void fake_units(int n) { units = n; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int attr, int dev) { (void)attr; (void)dev; *v = units; return 0; }
int hipMalloc(void** p, size_t n) { *p = malloc(n ? n : 1); return 0; }
int hipFree(void* p) { free(p); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* st) { (void)kind; (void)st; memcpy(d, s, n); return 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = &launches; return 0; }
int hipStreamSynchronize(void* s) { (void)s; return 0; }
int hipStreamIsCapturing(void* s, int* c) { (void)s; *c = 0; return 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { (void)f; *e = &launches; return 0; }
int hipEventRecord(void* e, void* s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(void* e) { (void)e; return 0; }
int hipEventDestroy(void* e) { (void)e; return 0; }
int hipGetLastError(void) { return 0; }
const char* hipGetErrorString(int e) { return e ? "stand-in error" : "no error"; }
typedef struct { unsigned x, y, z; } dim3_t;
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t s, void* st) { (void)g; (void)b; (void)s; (void)st; return 0; }
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* s, void** st) { g->x = g->y = g->z = b->x = b->y = b->z = 1; *s = 0; *st = 0; return 0; }
int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** a, size_t s, void* st) { (void)f; (void)g; (void)b; (void)a; (void)s; (void)st; ++launches; return 0; }
"""

PROGRAM = r"""
import ctypes, json, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
lengths, heads, d = json.loads(sys.argv[3]), int(sys.argv[4]), int(sys.argv[5])
cu = (ctypes.c_int32 * (len(lengths) + 1))(0)
for i, n in enumerate(lengths):
    cu[i + 1] = cu[i] + n
plan, p, i64, f32, size = ctypes.c_void_p(), ctypes.c_void_p, ctypes.c_int64, ctypes.c_float, ctypes.c_size_t
assert lib.hspmd_attn_plan_create(cu, len(lengths), heads, heads, d, p(0), ctypes.byref(plan)) == 0
lib.hspmd_attn_bwd_workspace_bytes.restype = size
lib.hspmd_last_error.restype = ctypes.c_char_p
need, buf, stride = lib.hspmd_attn_bwd_workspace_bytes(plan), p(1 << 20), i64(heads * d)
for units in (0, 256, 0):          # (the count is asked for until it has been answered, and then kept)
    fake.fake_units(units)
    before = fake.fake_launches()
    rc = lib.hspmd_attn_varlen_fwd(plan, buf, buf, buf, stride, stride, f32(0), buf, buf, p(0))
    forward = (rc, fake.fake_launches() - before)
    before = fake.fake_launches()
    rc = lib.hspmd_attn_varlen_bwd(plan, buf, buf, buf, buf, buf, buf, stride, stride, f32(0), buf, buf, buf, 0, buf, size(need), p(0))
    print(units, *forward, rc, fake.fake_launches() - before, (lib.hspmd_last_error() or b"").decode().replace(" ", "_") or "-")
"""

OK, ERR_HIP = 0, 4


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("hip_stand_in")
    src, so = tmp / "hip.c", tmp / "hip.so"
    src.write_text(STAND_IN)
    subprocess.run(["gcc", "-O1", "-Wall", "-shared", "-fPIC", "-o", str(so), str(src)], check=True)
    if not os.path.exists(lib_build.LIBRARY):
        lib_build.build()
    return str(so)


@pytest.mark.parametrize("lengths,heads,d", [([400] * 40, 8, 128),        # many short items: persistent dK/dV workgroups
                                             ([2048] * 4, 32, 128)])     # whole items, one workgroup each
def test_a_pass_that_cannot_be_sized_is_an_error(stand_in, lengths, heads, d):
    out = subprocess.run([sys.executable, "-c", PROGRAM, stand_in, lib_build.LIBRARY, json.dumps(lengths), str(heads), str(d)],
                         capture_output=True, text=True)
    assert out.returncode == 0, out.stderr[-2000:]
    unknown, known, kept = [line.split() for line in out.stdout.splitlines()]
    persistent = len(lengths) > 10
    assert unknown[1:3] == [str(ERR_HIP), "0"]                      # the forward is always persistent
    # a backward that reports success has launched both of its passes
    assert unknown[3:5] == ([str(ERR_HIP), "1"] if persistent else [str(OK), "2"]), unknown
    assert known[1:5] == kept[1:5] == [str(OK), "1", str(OK), "2"]
