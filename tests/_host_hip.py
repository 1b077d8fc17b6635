"""A stand-in for the HIP runtime on the CPU, for the library's host side: device memory is host memory, kernels are
logged and not run, allocations fail on demand.  Loaded with its symbols global before the library, whose own calls
then come here; a process that did so cannot use a GPU, so every scenario gets a child process of its own."""
import ctypes as C
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2311_15806_amd", "libpipe_hip.so")

SOURCE = r"""
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
typedef struct { uint32_t x, y, z; } grid_t;
typedef void (*launch_fn)(const char* name, uint32_t gx, uint32_t gy, uint32_t gz, uint32_t block, void** args);
static struct { const void* f; const char* name; } reg[4096];
static int n_reg;
static launch_fn on_launch;
static long mallocs, fail_at, launches, fail_launch;
static int capturing;
static grid_t cfg_g, cfg_b;
static size_t cfg_shmem;
static void* cfg_st;
void host_set(launch_fn f) { on_launch = f; }
void host_fail(long nth) { mallocs = 0; fail_at = nth; }     /* the nth allocation from now on fails; 0: none */
void host_fail_launch(long nth) { launches = 0; fail_launch = nth; }   /* the same of launches */
long host_mallocs(void) { return mallocs; }
void host_capture(int on) { capturing = on; }
void** __hipRegisterFatBinary(const void* d) { static void* h; (void)d; return &h; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* f, char* df, const char* name, unsigned t, void* a, void* b, void* c, void* d, int* w) {
  (void)m; (void)df; (void)t; (void)a; (void)b; (void)c; (void)d; (void)w;
  if (n_reg < 4096) { reg[n_reg].f = f; reg[n_reg++].name = name; }
}
void __hipRegisterVar(void** m, void* v, char* h, char* n, int e, size_t s, int c, int g) {
  (void)m; (void)v; (void)h; (void)n; (void)e; (void)s; (void)c; (void)g;
}
int __hipPushCallConfiguration(grid_t g, grid_t b, size_t s, void* st) { cfg_g = g; cfg_b = b; cfg_shmem = s; cfg_st = st; return 0; }
int __hipPopCallConfiguration(grid_t* g, grid_t* b, size_t* s, void** st) { *g = cfg_g; *b = cfg_b; *s = cfg_shmem; *st = cfg_st; return 0; }
static int last;
int hipLaunchKernel(const void* f, grid_t g, grid_t b, void** args, size_t s, void* st) {
  (void)s; (void)st;
  ++launches;
  if (fail_launch > 0 && launches == fail_launch) return last = 9;
  /* the runtime's limit: fewer than 2^32 threads in x */
  if (g.x == 0 || g.y == 0 || g.z == 0 || g.y > 65535 || g.z > 65535 || (uint64_t)g.x * b.x >= (1ull << 32)) return last = 9;
  for (int i = 0; i < n_reg; ++i)
    if (reg[i].f == f && on_launch) on_launch(reg[i].name, g.x, g.y, g.z, b.x, args);
  return 0;
}
int hipExtLaunchKernel(const void* f, grid_t g, grid_t b, void** args, size_t s, void* st, void* e0, void* e1, int fl) {
  (void)e0; (void)e1; (void)fl;
  return hipLaunchKernel(f, g, b, args, s, st);
}
int hipMalloc(void** p, size_t n) {
  ++mallocs;
  if (fail_at > 0 && mallocs == fail_at) return last = 2;
  *p = calloc(1, n ? n : 1);
  return *p ? 0 : (last = 2);
}
int hipFree(void* p) { free(p); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int k) {
  memcpy(d, s, n);
  if (k == 1 && on_launch) on_launch("hipMemcpy", (uint32_t)n, 1, 1, 1, &d);   /* to the device */
  return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { (void)k; (void)st; memcpy(d, s, n); return 0; }
int hipMemcpyToSymbol(const void* d, const void* s, size_t n, size_t o, int k) { (void)d; (void)s; (void)n; (void)o; (void)k; return 0; }
int hipMemset(void* d, int v, size_t n) {
  if (on_launch) on_launch("hipMemset", (uint32_t)n, 1, 1, 1, 0);
  memset(d, v, n);
  return 0;
}
int hipMemsetAsync(void* d, int v, size_t n, void* st) { (void)st; memset(d, v, n); return 0; }
int hipGetSymbolAddress(void** p, const void* sym) { static void* a; (void)sym; if (!a) a = calloc(1, 16 << 20); *p = a; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipStreamSynchronize(void* st) { (void)st; return capturing ? (last = 900) : 0; }
int hipStreamIsCapturing(void* st, int* s) { (void)st; *s = capturing; return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetLastError(void) { int l = last; last = 0; return l; }
const char* hipGetErrorString(int e) { return e == 2 ? "out of memory" : e == 9 ? "invalid configuration argument" : "error"; }
int hipFuncSetAttribute(const void* f, int a, int v) { (void)f; (void)a; (void)v; return 0; }
int hipEventCreate(void** e) { *e = calloc(1, 8); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void* e, void* st) { (void)e; (void)st; return 0; }
int hipEventSynchronize(void* e) { (void)e; return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 0; return 0; }
"""


class Runtime:
    """The stand-in and, bound to it, the library: `lib`.  `launches` logs (kernel, grid, arguments) in order."""

    def __init__(self, shim):
        self.host = C.CDLL(shim, mode=os.RTLD_GLOBAL | os.RTLD_NOW)
        self.host.host_fail.argtypes = self.host.host_fail_launch.argtypes = [C.c_long]
        self.host.host_mallocs.restype = C.c_long
        self.lib = C.CDLL(LIB)
        self.launches = []
        self.copied = []        # what was copied to the device synchronously (tables), in order
        self.kept = []          # what the next expansion's orders keep: lists of groups, order 2 first
        self._cb = C.CFUNCTYPE(None, C.c_char_p, *[C.c_uint32] * 4, C.POINTER(C.c_void_p))(self._launched)
        self.host.host_set(self._cb)

    def _launched(self, name, gx, gy, gz, block, args):
        name = name.decode()
        if name == "hipMemcpy":
            self.copied.append(C.string_at(args[0], gx))
            return
        self.launches.append((name, (gx, gy, gz), block))
        if "group_compact_kernel" in name:      # the selection's last launch (flags, groups, kept groups): the test's choice
            gids = C.cast(args[2], C.POINTER(C.POINTER(C.c_int32)))[0]
            for i, g in enumerate(self.kept.pop(0)):
                gids[i] = g

    def names(self):
        """The kernels launched since the last call."""
        out, self.launches = [l[0] for l in self.launches], []
        return out

    def expand(self, out, inp, bits, K, gamma, group, kept=()):
        self.kept = [list(k) for k in kept]
        W = (C.c_float * (out * inp))()
        h = C.c_void_p()
        self.lib.pipe_expand.argtypes = [C.c_void_p] + [C.c_int] * 4 + [C.c_float, C.c_int, C.c_void_p, C.POINTER(C.c_void_p)]
        rc = self.lib.pipe_expand(W, out, inp, bits, K, gamma, group, None, C.byref(h))
        assert rc == 0, rc
        self.names()
        return h


def run(script, scenario, tmp_path):
    """Runs `scenario` (a function of a Runtime) of the test file `script` in a process of its own."""
    src, shim = os.path.join(str(tmp_path), "host_hip.c"), os.path.join(str(tmp_path), "host_hip.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", shim, src], check=True)
    r = subprocess.run([sys.executable, script, scenario, shim], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
