"""A stand-in for the HIP runtime, for tests of the library's host paths without
a GPU: device memory is host memory, a kernel launch only notes the kernel's
name.  A program that loads it first (RTLD_GLOBAL) and the library after it runs
the library's own planning, uploads, routes and launch sequences; what a test
wants to go wrong (an allocation that fails, a stream under capture) is set
through its hh_ functions.  run() gives a program its own process."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <condition_variable>
#include <chrono>
#include <map>
#include <mutex>
#include <new>
#include <set>
#include <string>

namespace {
std::mutex mu;
std::condition_variable cv;
std::map<const void *, std::string> names;
std::map<const void *, std::pair<std::string, void *>> vars;
std::string log_;
thread_local int last_error = 0;
int capturing = 0, refused_in_capture = 0, fail_next = 0, n_malloc = 0;
int hold = 0, held = 0;
thread_local size_t throw_above = 0;
struct { unsigned x[6]; size_t sh; void *s; } cfg;
int err(int e) { last_error = e; return e; }
}

void *operator new(std::size_t n)
{
    if (throw_above && n >= throw_above)
        throw std::bad_alloc();
    void *p = std::malloc(n ? n : 1);
    if (!p)
        throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

extern "C" {
// ---- what a test sets and reads
void hh_capture(int on) { capturing = on; refused_in_capture = 0; }
int hh_refused_in_capture() { return refused_in_capture; }
void hh_fail_next(int n) { std::lock_guard<std::mutex> l(mu); fail_next = n; }
int hh_mallocs() { std::lock_guard<std::mutex> l(mu); return n_malloc; }
void hh_throw_above(size_t n) { throw_above = n; }   // of the calling thread; 0: never
int hh_last_error() { return last_error; }
// hipMalloc waits (20 s at most) until hh_hold(0); hh_held: a thread is waiting
void hh_hold(int on) { std::lock_guard<std::mutex> l(mu); hold = on; cv.notify_all(); }
int hh_held() { std::lock_guard<std::mutex> l(mu); return held; }
// names of the kernels launched since the last call, one a line
const char *hh_launches()
{
    static std::string out;
    std::lock_guard<std::mutex> l(mu);
    out.swap(log_);
    log_.clear();
    return out.c_str();
}

// ---- the runtime
void **__hipRegisterFatBinary(const void *) { static void *p; return &p; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *)
{
    names[f] = name;
}
void __hipRegisterVar(void **, void *var, char *, char *name, int, size_t size, int, int)
{
    vars[var] = {name, std::calloc(1, size)};
}
int __hipPushCallConfiguration(...) { return 0; }
int __hipPopCallConfiguration(void *, void *, size_t *sh, void **s) { *sh = 0; *s = nullptr; return 0; }
struct dim3_ { unsigned x, y, z; };
int hipLaunchKernel(const void *f, dim3_, dim3_, void **, size_t, void *)
{
    std::lock_guard<std::mutex> l(mu);
    log_ += names[f] + "\n";
    return 0;
}
int hipMalloc(void **p, size_t n)
{
    std::unique_lock<std::mutex> l(mu);
    ++n_malloc;
    if (hold) {
        ++held;
        cv.wait_for(l, std::chrono::seconds(20), [] { return !hold; });
        --held;
    }
    if (capturing) {
        ++refused_in_capture;
        return err(900);   // hipErrorStreamCaptureUnsupported
    }
    if (fail_next > 0) {
        --fail_next;
        return err(2);     // hipErrorOutOfMemory
    }
    *p = std::calloc(1, n);
    return 0;
}
int hipFree(void *p) { std::free(p); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int) { std::memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) { std::memcpy(d, s, n); return 0; }
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
const char *hipGetErrorString(int e) { return e == 2 ? "out of memory" : "error"; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int) { return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 160 * 1024; return 0; }
int hipDeviceSynchronize() { return 0; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipGetSymbolAddress(void **p, const void *var) { *p = vars[var].second; return 0; }
int hipEventCreate(void **e) { *e = std::malloc(1); return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { *e = std::malloc(1); return 0; }
int hipEventDestroy(void *e) { std::free(e); return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *t, void *, void *) { *t = 0.0f; return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { *s = std::malloc(1); return 0; }
int hipStreamDestroy(void *s) { std::free(s); return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
int hipStreamIsCapturing(void *, int *st) { *st = capturing ? 1 : 0; return 0; }
}
"""

# what every program starts with: hh (the stand-in), abi, and short names for
# calls on host buffers; each returns (status, kernels launched)
PRELUDE = r"""
import ctypes, sys
import numpy as np
hh = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
hh.hh_launches.restype = ctypes.c_char_p
hh.hh_throw_above.argtypes = [ctypes.c_size_t]
sys.path.insert(0, sys.argv[2])
from paper_2408_00836_amd import abi
L = abi.lib()

def buf(n):
    return ctypes.create_string_buffer(int(n))

def launched():
    return hh.hh_launches().decode().split()

def has(kernels, part):
    return any(part in k for k in kernels)

def out(st):
    return st, launched()

class Model:
    def __init__(self, nx, ny, layers, **kw):
        self.h, self.layers = abi.hubbard_create(nx, ny, **kw), layers
        self.np = abi.hubbard_param_count(self.h, layers)
        self.theta = np.linspace(0.1, 0.4, max(1, self.np))
        self.E, self.g = np.zeros(1), np.zeros(max(1, self.np))
        q = abi.hubbard_query(self.h)
        self.n_qubits = q["n_qubits"] if isinstance(q, dict) else q[0]
        self.vec = [buf(16 << self.n_qubits) for _ in range(2)]
        self.ws = {}

    def work(self, op):
        if op not in self.ws:
            self.ws[op] = buf(abi.hubbard_workspace_size(self.h, self.layers, op))
        return self.ws[op]

    def timing(self, on):
        abi.hubbard_set_timing(self.h, on)

    def energy_grad(self):
        w = self.work(abi.HUBBARD_OP_ENERGY_GRAD)
        return out(L.energy_grad(self.h, self.theta.ctypes.data, self.layers, self.E.ctypes.data,
                                 self.g.ctypes.data, ctypes.addressof(w), len(w), None))

    def energy(self):
        w = self.work(abi.HUBBARD_OP_ENERGY)
        return out(L.energy(self.h, self.theta.ctypes.data, self.layers, self.E.ctypes.data,
                            ctypes.addressof(w), len(w), None))

    def noalloc(self):
        return out(L.energy_grad_noalloc(self.h, self.theta.ctypes.data, self.layers,
                                         self.E.ctypes.data, self.g.ctypes.data, None))

    def prepare(self):
        return out(L.hubbard_prepare_state(self.h, self.theta.ctypes.data, self.layers,
                                           ctypes.addressof(self.vec[0]), None))

    def ansatz(self):
        return out(L.ansatz_apply(self.h, self.theta.ctypes.data, self.layers,
                                  ctypes.addressof(self.vec[0]), None))

    def apply_h(self):
        return out(L.hamiltonian_apply(self.h, ctypes.addressof(self.vec[0]),
                                       ctypes.addressof(self.vec[1]), None))

    def sector_eg(self):
        w = buf(abi.hubbard_sector_workspace_size(self.h, self.layers,
                                                  abi.HUBBARD_SECTOR_ENERGY_GRAD))
        return out(L.sector_energy_grad(self.h, self.theta.ctypes.data, self.layers,
                                        self.E.ctypes.data, self.g.ctypes.data,
                                        ctypes.addressof(w), len(w), None))

class Batch:
    def __init__(self, models):
        self.models = models
        n = len(models)
        self.h = (ctypes.c_void_p * n)(*[m.h for m in models])
        self.layers = (ctypes.c_int32 * n)(*[m.layers for m in models])
        off = np.concatenate([[0], np.cumsum([m.np for m in models])]).astype(np.int64)
        self.off = (ctypes.c_int64 * n)(*off[:n])
        self.theta = np.linspace(0.1, 0.4, int(off[n]) + 1)
        self.E, self.g = np.zeros(n), np.zeros(int(off[n]) + 1)
        self.need = abi.hubbard_batch_workspace_size([m.h for m in models],
                                                     [m.layers for m in models])
        self.ws = buf(self.need)

    def energy_grad(self, ws_bytes=None):
        return out(L.energy_grad_batch(self.h, len(self.models), self.theta.ctypes.data, self.off,
                                       self.layers, self.E.ctypes.data, self.g.ctypes.data,
                                       ctypes.addressof(self.ws), ws_bytes or self.need, None))
"""


def build(folder):
    src, lib = os.path.join(folder, "host_hip.cpp"), os.path.join(folder, "host_hip.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", src, "-o", lib], check=True)
    return lib


def run(lib, program, timeout=120):
    """Run PRELUDE + program in a process of its own; it fails by an assertion
    or any other error."""
    p = subprocess.run([sys.executable, "-c", PRELUDE + program, lib, ROOT], text=True,
                       capture_output=True, timeout=timeout)
    assert p.returncode == 0, f"exit {p.returncode}\n{p.stdout}\n{p.stderr}"
    return p.stdout
