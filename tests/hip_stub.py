"""Runs host code of the library without a GPU: a stand-in for the HIP runtime calls it makes (device
memory is host memory, launches are recorded and do nothing), preloaded into a subprocess. Covers plan
creation, schedules and launch shapes; no kernel runs."""

import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
typedef struct { uint32_t x, y, z; } dim3_t;
enum { MAXL = 4096 };
static struct { const void* f; dim3_t grid, block; size_t lds; } launches[MAXL];
static struct { dim3_t grid, block; size_t lds; void* s; } pushed;
static int n_launches, n_alloc, n_copy;
static size_t copied;
static float elapsed = 1.f, next_elapsed[MAXL];
static int n_elapsed, at_elapsed;
/* what the tests read */
void stub_reset(void) { n_launches = n_alloc = n_copy = 0; copied = 0; }
int stub_launches(void) { return n_launches; }
uint32_t stub_grid(int i) { return launches[i].grid.x; }
uint32_t stub_block(int i) { return launches[i].block.x; }
int stub_allocs(void) { return n_alloc; }
int stub_copies(void) { return n_copy; }
size_t stub_copied(void) { return copied; }
void stub_elapsed(const float* v, int n) { memcpy(next_elapsed, v, n * sizeof(float)); n_elapsed = n; at_elapsed = 0; }
const char* stub_kernel(int i) { Dl_info d; return dladdr(launches[i].f, &d) && d.dli_sname ? d.dli_sname : ""; }
/* the HIP runtime calls of the library */
int hipMalloc(void** p, size_t n) { ++n_alloc; *p = aligned_alloc(256, (n + 255) / 256 * 256); return *p ? 0 : 2; }
int hipFree(void* p) { free(p); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int k) { ++n_copy; copied += n; memcpy(d, s, n); return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { *v = 256; return 0; }
int hipGetDevicePropertiesR0600(void* p, int d) { memset(p, 0, 1472); return 0; }
int hipFuncSetAttribute(const void* f, int a, int v) { return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int b, size_t l) { *n = 1; return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipGetLastError(void) { return 0; }
const char* hipGetErrorString(int e) { return "stub"; }
int hipGetSymbolAddress(void** p, const void* s) { static char x[256]; *p = x; return 0; }
int hipEventCreate(void** e) { *e = malloc(1); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void* e, void* s) { return 0; }
int hipEventSynchronize(void* e) { return 0; }
int hipEventElapsedTime(float* t, void* a, void* b) {
  *t = at_elapsed < n_elapsed ? next_elapsed[at_elapsed++] : elapsed;
  return 0;
}
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, void* s) {
  pushed.grid = g; pushed.block = b; pushed.lds = lds; pushed.s = s; return 0;
}
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* lds, void** s) {
  *g = pushed.grid; *b = pushed.block; *lds = pushed.lds; *s = pushed.s; return 0;
}
int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** args, size_t lds, void* s) {
  if ((uint64_t)g.x * b.x >= (uint64_t)1 << 32 || !g.x) return 9; /* hipErrorInvalidConfiguration */
  if (n_launches < MAXL) { launches[n_launches].f = f; launches[n_launches].grid = g; launches[n_launches].block = b;
    launches[n_launches].lds = lds; ++n_launches; }
  return 0;
}
"""

PRELUDE = """
import ctypes, json, os, sys
sys.path.insert(0, {root!r})
import numpy as np
import synthgen
import paper_1103_4881_amd as aol
stub = ctypes.CDLL({lib!r})
stub.stub_kernel.restype = ctypes.c_char_p
stub.stub_copied.restype = ctypes.c_size_t
stub.stub_grid.restype = stub.stub_block.restype = ctypes.c_uint32
def launches():
    return [(stub.stub_kernel(i).decode(), stub.stub_grid(i), stub.stub_block(i)) for i in range(stub.stub_launches())]
BUF = 1 << 20  # an address that no call reads
"""


def run(tmp_path, script):
    """The JSON object that `script` prints last, run with the stand-in (fails if the process dies)."""
    src, lib = tmp_path / "hip_stub.c", tmp_path / "libhip_stub.so"
    if not lib.exists():
        src.write_text(SOURCE)
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-w", "-o", str(lib), str(src), "-ldl"], check=True)
    env = dict(os.environ, LD_PRELOAD=str(lib))
    r = subprocess.run([sys.executable, "-c", PRELUDE.format(root=ROOT, lib=str(lib)) + script], env=env, cwd=ROOT,
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, f"exit {r.returncode}\n{r.stdout}\n{r.stderr[-3000:]}"
    return json.loads(r.stdout.strip().splitlines()[-1])
