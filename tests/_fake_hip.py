"""A stand-in for the HIP runtime, for tests of the library's host side without a GPU: the built library runs in a child
process against a libamdhip64 that only records what is asked of it (kernels by name with their grid, allocations, kernel
attributes) and can refuse memory or attributes.  Nothing is executed; addresses are made up."""
import json
import os
import re
import subprocess
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_C = r"""
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3_t;
static char log_[1 << 22];
static size_t len_;
#define LOG(...) (len_ += (size_t)snprintf(log_ + len_, sizeof(log_) - len_, __VA_ARGS__))
static size_t limit_ = (size_t)-1, next_ = 1ull << 40;
static int capturing_, attr_fail_;
static struct { const void* host; char name[256]; } fn_[4096];
static int nfn_;
static dim3_t g_, b_; static size_t s_; static void* st_;

void fake_set(long long limit, int capturing, int attr_fail) {
  limit_ = limit < 0 ? (size_t)-1 : (size_t)limit; capturing_ = capturing; attr_fail_ = attr_fail; len_ = 0; log_[0] = 0;
}
const char* fake_log(void) { return log_; }
static const char* name_of(const void* f) {
  for (int i = 0; i < nfn_; ++i) if (fn_[i].host == f) return fn_[i].name;
  return "?";
}
void** __hipRegisterFatBinary(const void* d) { (void)d; static void* h; return &h; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned tl, void* a, void* b, void* c, void* d, int* w) {
  (void)m; (void)dev; (void)tl; (void)a; (void)b; (void)c; (void)d; (void)w;
  fn_[nfn_].host = host; snprintf(fn_[nfn_++].name, 256, "%s", name);
}
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t s, int c, int g) { (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g; }
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t s, void* st) { g_ = g; b_ = b; s_ = s; st_ = st; return 0; }
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* s, void** st) { *g = g_; *b = b_; *s = s_; *st = st_; return 0; }
int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** a, size_t s, void* st) {
  (void)a; (void)st; LOG("launch %s %u %u %zu\n", name_of(f), g.x, b.x, s); return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { (void)d; (void)s; (void)k; (void)st; LOG("copy %zu\n", n); return 0; }
int hipFuncSetAttribute(const void* f, int a, int v) {
  (void)a; int bad = attr_fail_ && strstr(name_of(f), "slab_conv3") != 0; LOG("attribute %s %d %d\n", name_of(f), v, bad); return bad ? 1 : 0;
}
int hipMalloc(void** p, size_t n) {
  int bad = n > limit_; LOG("malloc %zu %d\n", n, bad);
  if (bad) return 2;
  *p = (void*)next_; next_ += (n + 4095) / 4096 * 4096; return 0;
}
int hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = (void*)(1ull << 36); return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetDeviceCount(int* n) { *n = 1; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipGetLastError(void) { return 0; }
int hipStreamIsCapturing(void* st, int* c) { (void)st; *c = capturing_; return 0; }
"""

# what the child runs before the test's own lines: L (the library), T (a tensor), call(), events()
_PRELUDE = r"""
import ctypes, json, sys
L = ctypes.CDLL(sys.argv[1])
F = ctypes.CDLL("libamdhip64.so.7")
F.fake_set.argtypes = [ctypes.c_longlong, ctypes.c_int, ctypes.c_int]
F.fake_log.restype = ctypes.c_char_p
F32, BF16 = 0, 1
vp = ctypes.c_void_p
class T(ctypes.Structure):
    _fields_ = [("data", vp), ("n", ctypes.c_int32), ("h", ctypes.c_int32), ("w", ctypes.c_int32), ("c", ctypes.c_int32), ("dtype", ctypes.c_int32)]
L.lasnet_workspace_bytes.restype = ctypes.c_size_t
def call(entry, dtype, N, H, W, C, M, S, flags=0, stream=None, limit=-1, capturing=0, attr_fail=0, listed=True, ws=0, in_place=False):
    # one block call -> (status, events)
    F.fake_set(limit, capturing, attr_fail)
    size = 1 << 38
    x = T(vp(1 << 44).value, N, H, W, C, dtype)
    o = T(vp((1 << 44) + (0 if in_place else size)).value, N, H, W, C, dtype)
    p = [vp((1 << 45) + i * (1 << 36)) for i in range(8)]
    idx, count = (p[6], p[7]) if listed else (None, None)
    w = [p[0], p[1], p[2], p[3], p[4], p[5]]
    if entry == "planned":
        st = L.lasnet_sparse_bottleneck_planned(ctypes.byref(x), idx, count, None, S, M, p[0], p[1], p[3], p[5], ctypes.byref(o),
                                                flags, vp(1 << 43) if ws else None, ctypes.c_size_t(ws), vp(stream))
    elif entry == "packed":
        st = L.lasnet_sparse_bottleneck_packed(ctypes.byref(x), idx, count, S, M, p[0], p[1], p[3], p[5], ctypes.byref(o), flags, vp(stream))
    elif entry == "dense":
        st = L.lasnet_dense_bottleneck(ctypes.byref(x), M, *w, ctypes.byref(o), flags, vp(stream))
    else:
        f = L.lasnet_sparse_bottleneck_noalloc if entry == "noalloc" else L.lasnet_sparse_bottleneck_ex
        st = f(ctypes.byref(x), idx, count, S, M, *w, ctypes.byref(o), flags, vp(stream))
    return st, [l.split() for l in F.fake_log().decode().splitlines()]
def kernels(ev):
    return [e[1] for e in ev if e[0] == "launch"]
"""


def run(lines: str):
    """Runs `lines` (which assign to `result`) in a child process with the stand-in runtime; returns the result."""
    from paper_2210_06223_amd import build
    with tempfile.TemporaryDirectory() as d:
        src, ver = os.path.join(d, "fake.c"), os.path.join(d, "fake.map")
        with open(src, "w") as f:
            f.write(_C)
        with open(ver, "w") as f:
            f.write("hip_4.2 { *; };\nhip_4.3 { hipStreamIsCapturing; };\n")
        subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", os.path.join(d, "libamdhip64.so.7"), src,
                        "-Wl,-soname,libamdhip64.so.7", "-Wl,--version-script=" + ver], check=True)
        env = dict(os.environ, LD_LIBRARY_PATH=d + ":" + os.environ.get("LD_LIBRARY_PATH", ""))
        r = subprocess.run([sys.executable, "-c", _PRELUDE + lines + "\nprint('RESULT ' + json.dumps(result))", build.LIB], env=env,
                           capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        return json.loads(r.stdout.split("RESULT ")[1])


def kernel_name(mangled: str) -> str:
    """"slab_conv2_kernel<256,1,2,1>" from a mangled template kernel of the library (integer and type arguments)."""
    m = re.search(r"GLOBAL__N_1\d+([a-z]\w*?_kernel)(I.*?EE)?", mangled)
    args = re.findall(r"L[ib](\d+)E|NS\d*_\d*([A-Z]\w*?)E", m.group(2) or "")
    return m.group(1) + ("<" + ",".join(a or re.sub(r"^\d+", "", b) for a, b in args) + ">" if args else "")
