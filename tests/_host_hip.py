"""The library on a HIP runtime of the host: device memory is host memory, a
kernel launch is recorded by name and grid and does not run. For tests of the
planner, the launch plan and error paths (a call that fails half way) without a
GPU. The stub is loaded with its symbols global, ahead of the library, in a
process of its own.
"""
import json
import os
import re
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STUB = r"""
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
typedef struct { uint32_t x, y, z; } dim3;
static struct { const void* f; const char* name; } fns[1024];
static int n_fns, pinned, device, memsets, fail_memset = -1;
static char log_buf[1 << 20];
static size_t log_len;
static dim3 cfg_g, cfg_b;
static size_t cfg_s;
static void* cfg_st;
/* for the tests */
int stub_pinned(void) { return pinned; }
int stub_device(void) { return device; }
void stub_fail_memset(int nth) { memsets = 0; fail_memset = nth; }
const char* stub_log(void) { log_buf[log_len] = 0; log_len = 0; return log_buf; }
/* registration and launches */
void** __hipRegisterFatBinary(const void* d) { static void* m; return &m; }
void __hipUnregisterFatBinary(void** m) {}
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned l, void* a, void* b, void* c, void* d, int* e) {
  fns[n_fns].f = host;
  fns[n_fns++].name = name;
}
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t s, int c, int g) {}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, void* st) { cfg_g = g; cfg_b = b; cfg_s = s; cfg_st = st; return 0; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, void** st) { *g = cfg_g; *b = cfg_b; *s = cfg_s; *st = cfg_st; return 0; }
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, void* st) {
  for (int i = 0; i < n_fns; ++i)
    if (fns[i].f == f && log_len + 512 < sizeof(log_buf))
      log_len += snprintf(log_buf + log_len, 512, "%s %u %u %zu %llu\n", fns[i].name, g.x, b.x, lds,
                          (unsigned long long)*(uintptr_t*)args[0]);
  return 0;
}
/* memory */
int hipMalloc(void** p, size_t n) { *p = calloc(n, 1); device += *p != 0; return *p ? 0 : 2; }
int hipFree(void* p) { device -= p != 0; free(p); return 0; }
int hipHostMalloc(void** p, size_t n, unsigned f) { *p = calloc(n, 1); pinned += *p != 0; return *p ? 0 : 2; }
int hipHostFree(void* p) { pinned -= p != 0; free(p); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { memcpy(d, s, n); return 0; }
int hipMemsetAsync(void* d, int v, size_t n, void* st) { if (memsets++ == fail_memset) return 1; memset(d, v, n); return 0; }
int hipGetSymbolAddress(void** p, const void* s) { static char a[32 << 20]; *p = a; return 0; }
/* the rest does nothing */
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipSetDevice(int d) { return 0; }
int hipGetLastError(void) { return 0; }
const char* hipGetErrorString(int e) { return "stub error"; }
int hipFuncSetAttribute(const void* f, int a, int v) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { *s = malloc(1); return 0; }
int hipStreamDestroy(void* s) { free(s); return 0; }
int hipStreamSynchronize(void* s) { return 0; }
int hipStreamBeginCapture(void* s, int m) { return 0; }
int hipStreamEndCapture(void* s, void** g) { *g = malloc(1); return 0; }
int hipGraphInstantiate(void** e, void* g, void* n, char* l, size_t s) { *e = malloc(1); return 0; }
int hipGraphLaunch(void* e, void* s) { return 0; }
int hipGraphDestroy(void* g) { free(g); return 0; }
int hipGraphExecDestroy(void* e) { free(e); return 0; }
int hipEventCreate(void** e) { *e = malloc(1); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void* e, void* s) { return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { *ms = 0; return 0; }
"""

PRELUDE = """
import ctypes, json, sys
sys.path[:0] = [%r, %r]
stub = ctypes.CDLL(%r, mode=ctypes.RTLD_GLOBAL)
stub.stub_log.restype = ctypes.c_char_p
import numpy as np
from paper_2408_01331_amd import unifiednn as U
from paper_2408_01331_amd import workloads as W
U.lib()


class Gemm(ctypes.Structure):  # the first fields of a grouped-GEMM problem
    _fields_ = [(k, ctypes.c_int64) for k in ("A", "B", "lda", "ldb")] + [(k, ctypes.c_int32) for k in (
        "M", "N", "K", "epi", "relu", "amode", "bmode", "tiles_n", "nsplit", "bias_tile", "model")] + [
        ("C", ctypes.c_int64), ("ldc", ctypes.c_int64)]


def launches():
    # (kernel, workgroups, threads, dynamic LDS, first argument) per launch since the last call
    return [[l.split()[0]] + [int(v) for v in l.split()[1:]] for l in stub.stub_log().decode().splitlines()]


def gemm_of(launch):
    # the first problem of a grouped-GEMM launch
    return Gemm.from_address(launch[4])
"""


def run(code, tmp_path):
    """Run `code` (which has `U`, `W`, `np`, `stub`, `launches()` on the stub
    and `gemm_of()`) on the stub and return the value it assigns to `result`."""
    src, so = str(tmp_path / "stub.c"), str(tmp_path / "stub.so")
    if not os.path.exists(so):
        with open(src, "w") as f:
            f.write(STUB)
        subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-w", src, "-o", so], check=True)
    prog = PRELUDE % (ROOT, os.path.dirname(os.path.abspath(__file__)), so) + code + \
        "\nprint('RESULT ' + json.dumps(result))\n"
    r = subprocess.run([sys.executable, "-c", prog], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    return json.loads([l for l in r.stdout.splitlines() if l.startswith("RESULT ")][-1][7:])


def gemm_variants(log):
    """Per grouped-GEMM launch of a recorded step: (backward, tile variant)."""
    out = []
    for name, *_ in log:
        m = re.search(r"gemm_kernelI[tf]Li(\d)ELb[01]ELb([01])E", name)
        if m:
            out.append((m.group(2) == "1", int(m.group(1))))
    return out
