"""The library on a stand-in for the HIP runtime: device memory is host memory, kernels are not run,
and every launch, copy and allocation is written down.  For tests of what the host side does (which
kernels a call launches, what an error path gives back) that need no GPU.

run(script, tmp_path) runs `script` in a process of its own, in which `calls` is the stand-in (a
CDLL), `lib` the library, `lbm` its binding, `W` the workloads, and log() returns the names of the
calls since the last log(): "launch <kernel>", "copy", "set" or "host alloc <the thread's capture
mode>" (0 global, 2 relaxed)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cxxabi.h>
#include <dlfcn.h>
#include <cstdlib>
#include <cstring>
#include <new>
#include <string>
#include <utility>
struct dim3 { unsigned x, y, z; };
static std::string text;
static int left_copies = -1, left_allocs = -1;      // calls until one fails, -1: none does
static int mode = 0, capturing = 0;
static dim3 g_grid, g_block;
static bool failing(int &n) { return n >= 0 && n-- == 0; }
static int left_news = -1;
static bool own = false;        // the stand-in's own allocations
void *operator new(size_t n)
{
    void *p = left_news == 0 && !own ? nullptr : malloc(n ? n : 1);
    if (left_news > 0 && !own) --left_news;
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }
static void note(const std::string &s) { text += s + "\n"; }
#define OK(name) int name() { return 0; }
extern "C" {
const char *calls_text() { return text.c_str(); }
void calls_clear() { text.clear(); }
void calls_fail_new(int n) { text.reserve(1 << 16); left_news = n; }      // that many succeed, then none (-1: all)
void calls_fail_copy(int n) { left_copies = n; }
void calls_fail_alloc(int n) { left_allocs = n; }
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t, void *) { g_grid = g; g_block = b; return 0; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, void **st) { *g = g_grid; *b = g_block; *s = 0; *st = nullptr; return 0; }
int hipLaunchKernel(const void *f, dim3, dim3, void **, size_t, void *)
{
    Dl_info i;
    own = true;
    if (!dladdr(f, &i) || !i.dli_sname) i.dli_sname = "::?";
    int st;
    char *n = abi::__cxa_demangle(i.dli_sname, nullptr, nullptr, &st);
    const std::string s = st == 0 ? n : i.dli_sname;
    const size_t a = s.rfind("::", s.find('<')) + 2;
    note("launch " + s.substr(a, s.find_first_of("<(", a) - a));
    free(n);
    own = false;
    return 0;
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *)
{
    note("copy");
    if (failing(left_copies)) return 1;
    memcpy(d, s, n);
    return 0;
}
int hipMemsetAsync(void *d, int v, size_t n, void *) { note("set"); memset(d, v, n); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned)
{
    own = true;
    note("host alloc " + std::to_string(mode));
    own = false;
    if (failing(left_allocs)) return 2;
    *p = calloc(1, n);
    return 0;
}
int hipThreadExchangeStreamCaptureMode(int *m) { std::swap(*m, mode); return 0; }
int calls_mode() { return mode; }
void calls_capturing(int on) { capturing = on; }
int hipStreamIsCapturing(void *, int *status) { *status = capturing; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetSymbolAddress(void **p, const void *) { *p = calloc(1, 1 << 22); return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 1.0f; return 0; }
const char *hipGetErrorString(int) { return "stand-in error"; }
int hipEventCreate(void **e) { *e = e; return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { *e = e; return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { *s = s; return 0; }
int hipGraphCreate(void **g, unsigned) { *g = g; return 0; }
int hipGraphAddKernelNode(void **n, void *, const void *, size_t, const void *) { *n = n; return 0; }
int hipGraphInstantiate(void **e, void *, void *, char *, size_t) { *e = e; return 0; }
OK(hipEventDestroy) OK(hipEventRecord) OK(hipEventSynchronize) OK(hipGetLastError) OK(hipGraphDestroy)
OK(hipGraphExecDestroy) OK(hipGraphLaunch) OK(hipStreamDestroy) OK(hipStreamSynchronize) OK(hipStreamWaitEvent)
}
"""

PRELUDE = r"""
import ctypes as C, sys
sys.path.insert(0, {root!r})
calls = C.CDLL({so!r}, mode=C.RTLD_GLOBAL)
calls.calls_text.restype = C.c_char_p
import workloads as W
from paper_1505_02976_amd import lbm
lib = lbm.lib()
def log():
    t = calls.calls_text().decode().splitlines()
    calls.calls_clear()
    return t
def memory(n):
    b = C.create_string_buffer(int(n) + 256)
    return b, C.c_void_p((C.addressof(b) + 255) // 256 * 256)
class Sim:
    def __init__(self, cfg):
        p = lbm.make_params(cfg)
        n = lib.lbm_workspace_bytes(C.byref(p))
        self.keep, ws = memory(n)
        self.h = C.c_void_p()
        lbm._check(lib.lbm_init(C.byref(p), ws, n, None, C.byref(self.h)))
    def step(self, n):
        log()
        lbm._check(lib.lbm_step(self.h, n))
        return log()
class Batch:
    def __init__(self, cfgs):
        p = (lbm._Params * len(cfgs))(*[lbm.make_params(c) for c in cfgs])
        n = lib.lbm_batch_workspace_bytes(p, len(cfgs))
        self.keep, ws = memory(n)
        self.h = C.c_void_p()
        lbm._check(lib.lbm_batch_init(p, len(cfgs), ws, n, None, C.byref(self.h)))
    def step(self, n):
        log()
        lbm._check(lib.lbm_batch_step(self.h, n))
        return log()
"""


def run(script, tmp_path):
    src, so = str(tmp_path / "calls.cpp"), str(tmp_path / "calls.so")
    with open(src, "w") as fh:
        fh.write(SOURCE)
    subprocess.run(["g++", "-O1", "-w", "-shared", "-fPIC", "-o", so, src, "-ldl"], check=True)
    p = subprocess.run([sys.executable, "-c", PRELUDE.format(root=ROOT, so=so) + script], capture_output=True, text=True,
                       timeout=120)
    assert p.returncode == 0, p.stdout + p.stderr
    return p.stdout
