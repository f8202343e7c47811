"""The library on a stand-in for the HIP runtime that writes down what it is asked to do (no GPU).

Device memory is host memory, kernels are named and not run.  `record(program)` runs a Python program in a process of its own in
which `lib` is the library, `fake` the stand-in and `Plan` / `BlockPlan` make plans; what the program passes to `out` comes back."""
import json
import os
import re
import subprocess
import sys

from paper_2504_20490_amd import build as lib_build

STAND_IN = r"""
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
static char text[1 << 20];      /* one line per call that is recorded */
static size_t used;
static struct { const void* stub; const char* name; } kernels[4096];
static int count;
static unsigned grid[3];
static void line(const char* what, const char* more, unsigned n) {
    if (used + 512 + strlen(more) < sizeof text) used += (size_t)sprintf(text + used, "%s %s %u\n", what, more, n);
}
const char* fake_calls(void) { return text; }
void fake_forget(void) { used = 0; text[0] = 0; }
int fake_kernels(int i, const char** name) { if (i < count) *name = kernels[i].name; return count; }
void __hipRegisterFunction(void** m, const void* stub, char* dev, const char* name, unsigned lim, void* a, void* b, void* c, void* d, int* w) {
    (void)m; (void)dev; (void)lim; (void)a; (void)b; (void)c; (void)d; (void)w;
    if (count < 4096) { kernels[count].stub = stub; kernels[count++].name = strdup(name); }
}
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipSetDevice(int d) { (void)d; return 0; }
int hipDeviceGetAttribute(int* v, int attr, int dev) { (void)attr; (void)dev; *v = 256; return 0; }
int hipDeviceSynchronize(void) { line("sync", "device", 0); return 0; }
int hipMalloc(void** p, size_t n) { *p = malloc(n ? n : 1); line("malloc", "-", (unsigned)n); return 0; }
int hipFree(void* p) { free(p); line("free", "-", 0); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* st) { (void)kind; (void)st; memcpy(d, s, n); line("copy", "-", (unsigned)n); return 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = &count; return 0; }
int hipStreamSynchronize(void* s) { (void)s; return 0; }
int hipStreamIsCapturing(void* s, int* c) { (void)s; *c = 0; return 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { *e = malloc(1); line("event", "-", f); return 0; }
int hipEventRecord(void* e, void* s) { (void)e; (void)s; line("mark", "-", 0); return 0; }
int hipEventSynchronize(void* e) { (void)e; line("wait", "-", 0); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = (void*)(1 << 20); return 0; }
int hipGetLastError(void) { return 0; }
const char* hipGetErrorString(int e) { return e ? "stand-in error" : "no error"; }
typedef struct { unsigned x, y, z; } dim3_t;
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t s, void* st) { (void)b; (void)s; (void)st; grid[0] = g.x; return 0; }
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* s, void** st) { g->x = grid[0]; g->y = g->z = b->x = b->y = b->z = 1; *s = 0; *st = 0; return 0; }
int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** a, size_t s, void* st) {
    int i; (void)b; (void)a; (void)s; (void)st;
    for (i = 0; i < count && kernels[i].stub != f; ++i) {}
    line("launch", i < count ? kernels[i].name : "?", g.x);
    return 0;
}
"""

PRELUDE = r"""
import ctypes, json, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
args = json.loads(sys.argv[3])
fake.fake_calls.restype = ctypes.c_char_p
lib.hspmd_attn_bwd_workspace_bytes.restype = ctypes.c_size_t
p, i64, f32 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_float
ints = lambda a: (ctypes.c_int32 * max(len(a), 1))(*a)
def cu(lengths):
    ends = [0]
    for n in lengths:
        ends.append(ends[-1] + n)
    return ints(ends)
def calls():
    lines = [l.split() for l in fake.fake_calls().decode().splitlines()]
    fake.fake_forget()
    return [(a, b, int(c)) for a, b, c in lines]
class Plan:
    def __init__(self, lengths, hq, hkv, d):
        self.h, self.hq, self.hkv, self.d = p(), hq, hkv, d
        assert lib.hspmd_attn_plan_create(cu(lengths), len(lengths), hq, hkv, d, p(0), ctypes.byref(self.h)) == 0
    def update(self, lengths):
        assert lib.hspmd_attn_plan_update(self.h, cu(lengths), len(lengths)) == 0
    def forward(self):
        b, qs, ks = p(1 << 20), i64(self.hq * self.d), i64(self.hkv * self.d)
        assert lib.hspmd_attn_varlen_fwd(self.h, b, b, b, qs, ks, f32(0), b, b, p(0)) == 0
    def backward(self, workspace_bytes=None):
        b, qs, ks = p(1 << 20), i64(self.hq * self.d), i64(self.hkv * self.d)
        n = ctypes.c_size_t(workspace_bytes or lib.hspmd_attn_bwd_workspace_bytes(self.h))
        assert lib.hspmd_attn_varlen_bwd(self.h, b, b, b, b, b, b, qs, ks, f32(0), b, b, b, 0, b, n, p(0)) == 0
    def backward_static(self):
        b, qs, ks = p(1 << 20), i64(self.hq * self.d), i64(self.hkv * self.d)
        assert lib.hspmd_attn_varlen_bwd_static_ws(self.h, b, b, b, b, b, b, qs, ks, f32(0), b, b, b, 0, p(0)) == 0
    def destroy(self):
        assert lib.hspmd_attn_plan_destroy(self.h) == 0
class BlockPlan(Plan):
    def __init__(self, ql, kl, qp, kp, hq, hkv, d):
        self.h, self.hq, self.hkv, self.d = p(), hq, hkv, d
        assert lib.hspmd_attn_block_plan_create(cu(ql), cu(kl), ints(qp), ints(kp), len(ql), hq, hkv, d, p(0), ctypes.byref(self.h)) == 0
    def update(self, ql, kl, qp, kp):
        assert lib.hspmd_attn_block_plan_update(self.h, cu(ql), cu(kl), ints(qp), ints(kp), len(ql)) == 0
    def forward(self):
        b, qs, ks = p(1 << 20), i64(self.hq * self.d), i64(self.hkv * self.d)
        assert lib.hspmd_attn_block_fwd(self.h, b, b, b, qs, ks, f32(0), b, b, p(0)) == 0
    def backward(self):
        b, qs, ks = p(1 << 20), i64(self.hq * self.d), i64(self.hkv * self.d)
        n = ctypes.c_size_t(lib.hspmd_attn_bwd_workspace_bytes(self.h))
        assert lib.hspmd_attn_block_bwd(self.h, b, b, b, b, b, b, qs, ks, f32(0), b, 0, b, b, 0, b, n, p(0)) == 0
def out(x):
    print("OUT " + json.dumps(x))
"""


def build_stand_in(folder) -> str:
    src, so = folder / "recorder.c", folder / "recorder.so"
    src.write_text(STAND_IN)
    subprocess.run(["gcc", "-O1", "-Wall", "-shared", "-fPIC", "-o", str(so), str(src)], check=True)
    if not os.path.exists(lib_build.LIBRARY):
        lib_build.build()
    return str(so)


def record(stand_in: str, program: str, *args):
    run = subprocess.run([sys.executable, "-c", PRELUDE + program, stand_in, lib_build.LIBRARY, json.dumps(args)],
                         capture_output=True, text=True)
    assert run.returncode == 0, run.stderr[-2000:]
    return [json.loads(l[4:]) for l in run.stdout.splitlines() if l.startswith("OUT ")]


def kernel(mangled: str):
    """(name, template arguments) of a kernel of this library: its numbers, then TwoTeams and HeadPieces by name where they are among
    them, then whether its list is in the launch's arguments."""
    m = re.match(r"_ZN5hspmd(\d+)", mangled)
    if not m:
        return mangled, ()
    at = m.end() + int(m.group(1))
    values = re.match(r"I((?:L[ib]\d+E)*)(J(.*?)E)?", mangled[at:])
    if not values:
        return mangled[m.end():at], ()
    found = tuple(int(x) if t == "i" else x == "1" for t, x in re.findall(r"L([ib])(\d+)E", values.group(1)))
    if values.group(2) is None:
        return mangled[m.end():at], found
    pack = mangled[at:at + values.end() + 20]
    return mangled[m.end():at], found + tuple(x for x in ("TwoTeams", "HeadPieces") if x in pack) + ("InlineList" in pack,)
