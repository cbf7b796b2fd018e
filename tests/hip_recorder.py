"""The library's host side without a GPU: a recording HIP runtime.

`run(script)` runs a Python script in a process of its own where libmcc_hip.so
is bound to a small C++ stand-in for the HIP runtime.  Device memory there is
host memory, kernels do nothing but enter the log (except the front kernels,
whose cell lists the host reads back: they are worked out in C++), and the log
tells streams, events, allocations and launches in order.  The script gets

  L              the library (typed as native.load types it)
  np, native     numpy and the binding module
  Pop(sizes)     a population of cells of these sizes, one species; .args of
                 the sorted entry points
  ctx()          a new context
  log()          the log since the last call, as a list of dicts
  rt             the stand-in: rt.rec_malloc_limit(bytes) makes larger
                 allocations fail, rt.rec_fail_launch(k) the k-th launch from
                 here (from 1)

and what it prints comes back as the result (JSON by its last line)."""
import json
import os
import subprocess
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUNTIME = r"""
#include <hip/hip_runtime_api.h>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

static std::map<const void *, std::string> &kernels() {
  static std::map<const void *, std::string> k;
  return k;
}
static std::map<const void *, std::pair<size_t, void *>> &vars() {
  static std::map<const void *, std::pair<size_t, void *>> v;
  return v;
}
static std::vector<std::string> lines;
static std::map<const void *, int> ids;
static size_t limit = ~(size_t)0;
static int fail_launch;
static hipError_t last_error = hipSuccess;
static int id(const void *p) {
  if (!p) return 0;
  auto it = ids.find(p);
  return it != ids.end() ? it->second : (ids[p] = (int)ids.size() + 1);
}
static void put(const std::string &s) { lines.push_back(s); }
static std::string num(const char *k, long long v) {
  return std::string(", \"") + k + "\": " + std::to_string(v);
}
static std::string op(const char *o) { return std::string("{\"op\": \"") + o + "\""; }

// the cell lists of the front kernels
static void front(void **a, bool one) {
  const int64_t *off = *(const int64_t **)a[0];
  const int32_t n_cells = *(int32_t *)a[1], S = *(int32_t *)a[2];
  int32_t *lists = *(int32_t **)a[one ? 5 : 6];
  uint32_t *counts = *(uint32_t **)a[one ? 6 : 7];
  const int first = *(int *)a[one ? 11 : 9];
  static const int cap[7] = {128, 256, 512, 1024, 2048, 4096, 32768};
  memset(counts, 0, 7 * sizeof(uint32_t));
  for (int32_t c = 0; c < n_cells; ++c) {
    const int64_t m = off[(int64_t)(c + 1) * S] - off[(int64_t)c * S];
    if (m <= 0) continue;
    int b = first;
    while (b < 7 && m > cap[b]) ++b;
    if (b < 7) lists[(int64_t)b * n_cells + counts[b]++] = c;
  }
}

extern "C" {
int rec_log(char *buf, size_t len) {
  std::string s = "[";
  for (size_t i = 0; i < lines.size(); ++i) s += (i ? ", " : "") + lines[i] + "}";
  s += "]";
  if (s.size() + 1 > len) return -1;
  memcpy(buf, s.c_str(), s.size() + 1);
  lines.clear();
  return 0;
}
void rec_malloc_limit(size_t n) { limit = n; }
void rec_fail_launch(int k) { fail_launch = k; }

void **__hipRegisterFatBinary(const void *) { static void *m; return &m; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, uint3 *,
                           uint3 *, dim3 *, dim3 *, int *) {
  kernels()[host] = name;
}
void __hipRegisterVar(void **, void *var, char *, char *, int, size_t size, int, int) {
  vars()[var] = {size, nullptr};
}
static dim3 g_grid, g_block;
static size_t g_shared;
static hipStream_t g_stream;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st) {
  g_grid = g, g_block = b, g_shared = s, g_stream = st;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, hipStream_t *st) {
  *g = g_grid, *b = g_block, *s = g_shared, *st = g_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **a, size_t, hipStream_t s) {
  const std::string n = kernels()[f];
  if (fail_launch > 0 && --fail_launch == 0) {
    put(op("failed") + ", \"kernel\": \"" + n + "\"");
    return last_error = hipErrorInvalidConfiguration;
  }
  put(op("launch") + ", \"kernel\": \"" + n + "\"" + num("stream", id(s)) + num("grid", g.x) +
      num("block", b.x));
  if (n.find("k_front_one") != std::string::npos) front(a, true);
  else if (n.find("7k_frontE") != std::string::npos) front(a, false);
  return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) {
  put(op("malloc") + num("bytes", (long long)n) + num("ok", n <= limit));
  *p = n <= limit ? malloc(n ? n : 1) : nullptr;
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemset(void *p, int v, size_t n) { memset(p, v, n); return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *s) {
  auto &v = vars()[s];
  if (!v.second) v.second = calloc(1, v.first ? v.first : 1);
  *p = v.second;
  return hipSuccess;
}
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
  memset(p, 0, sizeof(*p));
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipGetLastError(void) {
  const hipError_t e = last_error;
  last_error = hipSuccess;
  return e;
}
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
  *n = 2;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  *s = (hipStream_t)malloc(1);
  put(op("stream") + num("id", id(*s)));
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { ids.erase(s); free(s); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
  *e = (hipEvent_t)malloc(1);
  put(op("event") + num("id", id(*e)));
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { ids.erase(e); free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  put(op("record") + num("event", id(e)) + num("stream", id(s)));
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  put(op("wait") + num("event", id(e)) + num("stream", id(s)));
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
  *s = hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
  *g = (hipGraph_t)malloc(1);
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t) {
  *x = (hipGraphExec_t)malloc(1);
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g) { free(g); return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) { free(x); return hipSuccess; }
}
"""

CHILD = r"""
import ctypes as C, json, os, sys, types
import numpy as np
rt = C.CDLL(sys.argv[1], C.RTLD_GLOBAL)
rt.rec_malloc_limit.argtypes = [C.c_size_t]
rt.rec_log.argtypes = [C.c_char_p, C.c_size_t]
sys.path.insert(0, sys.argv[2])
sys.modules["torch"] = types.ModuleType("torch")  # (the binding loads torch's HIP runtime with it)
from paper_2407_19151_amd import native
L = native.load()
_buf = C.create_string_buffer(1 << 24)

def log():
    assert rt.rec_log(_buf, len(_buf)) == 0
    return json.loads(_buf.value.decode())

class Pop:
    def __init__(self, sizes, collisions=((0, 0),)):
        self.n_cells, self.n = len(sizes), int(np.sum(sizes))
        self.offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        self.w = np.ones(self.n)
        self.v = np.zeros((3, self.n))
        self.t = np.zeros((3, self.n))
        self.sp, self.co = native._species([1.0], [-1.0]), native._collisions(collisions)
        self.nco = len(collisions)
    def _p(self, a):
        return a.ctypes.data
    def head(self):
        return [self.n, self.n_cells, 1, self._p(self.offsets), self._p(self.w)]
    def vel(self, a):
        return [self._p(a[i]) for i in range(3)]
    def tail(self):
        return [None, 1.0, self.sp, self.nco, self.co, 0.1, 10.0]

def ctx():
    h = C.c_void_p()
    assert L.mcc_create(C.byref(h), 0, None) == 0
    return h

def sorted_step(h, p, params=None):
    return L.mcc_collide_sorted(h, *p.head(), *p.vel(p.v), *p.tail(), 7, 0,
                                C.byref(params or native.make_params()), None, None)

def jvp(h, p, params=None):
    return L.mcc_collide_sorted_jvp(h, *p.head(), *p.vel(p.v), *p.vel(p.t), *p.tail(), 0.0, 7, 0,
                                    C.byref(params or native.make_params()), 0, None)

def adjoint(h, p, params=None):
    return L.mcc_collide_adjoint(h, *p.head(), *p.vel(p.v), *p.vel(p.t), *p.tail(), 7, 0,
                                 C.byref(params or native.make_params()), None)

def plan(h, p, params=None):
    q = C.c_void_p()
    rc = L.mcc_plan_create(h, C.byref(q), *p.head(), *p.vel(p.v), *p.tail(), 7,
                           C.byref(params or native.make_params()), None, None, 0)
    return rc, q

def collide(h, n, n_cells, params=None):
    p = Pop([n])
    cells, species = np.zeros(n, np.int32), np.zeros(n, np.int32)
    return L.mcc_collide(h, n, cells.ctypes.data, species.ctypes.data, n_cells, 1,
                         p.w.ctypes.data, *p.vel(p.v), *p.tail(), 7, 0,
                         C.byref(params or native.make_params()), None, None)

def steps(lines, name="collide_kernel"):
    return [x for x in lines if x["op"] == "launch" and name in x["kernel"]]

"""


def build(folder):
    """The stand-in as a shared library in `folder`."""
    src, lib = os.path.join(folder, "rt.cpp"), os.path.join(folder, "rt.so")
    open(src, "w").write(RUNTIME)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-w",
                    "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", src, "-o", lib], check=True)
    return lib


def run(lib, script):
    r = subprocess.run([sys.executable, "-c", CHILD + script, lib, ROOT], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-4000:]
    return json.loads(r.stdout.strip().splitlines()[-1])
