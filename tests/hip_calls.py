"""Runs a snippet in a process of its own whose HIP calls are counted.

A small library that defines hipMalloc, hipLaunchKernel and hipExtLaunchKernel is opened with
its symbols global before anything else, so libmagpie's references bind to it; it passes every
call on and keeps a trace ('m' allocation, 'k' launch, 't' timed launch) from calls.start() to
calls.stop().  calls.refuse(n): allocations of exactly n bytes fail as on a full device.
"""

import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>
typedef struct { unsigned x, y, z; } dim3_t;
static char trace[1 << 20];
static int length, on;
static size_t refused;
static void* real(const char* name) {
  void* lib = dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD);
  return dlsym(lib, name);
}
static void note(char c) {
  if (on && length < (int)sizeof(trace) - 1) trace[length++] = c;
}
int hipMalloc(void** p, size_t n) {
  static int (*f)(void**, size_t);
  if (!f) f = (int (*)(void**, size_t))real("hipMalloc");
  note('m');
  return f(p, refused && n == refused ? (size_t)1 << 60 : n);
}
int hipLaunchKernel(const void* k, dim3_t g, dim3_t b, void** a, size_t s, void* q) {
  static int (*f)(const void*, dim3_t, dim3_t, void**, size_t, void*);
  if (!f) f = (int (*)(const void*, dim3_t, dim3_t, void**, size_t, void*))real("hipLaunchKernel");
  note('k');
  return f(k, g, b, a, s, q);
}
int hipExtLaunchKernel(const void* k, dim3_t g, dim3_t b, void** a, size_t s, void* q, void* e0, void* e1, int fl) {
  static int (*f)(const void*, dim3_t, dim3_t, void**, size_t, void*, void*, void*, int);
  if (!f) f = (int (*)(const void*, dim3_t, dim3_t, void**, size_t, void*, void*, void*, int))real("hipExtLaunchKernel");
  note('t');
  return f(k, g, b, a, s, q, e0, e1, fl);
}
void calls_start(void) { length = 0; on = 1; }
const char* calls_stop(void) { on = 0; trace[length] = 0; return trace; }
void calls_refuse(size_t n) { refused = n; }
"""

PRELUDE = r"""
import ctypes, json, sys
shim = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
shim.calls_stop.restype = ctypes.c_char_p
shim.calls_refuse.argtypes = [ctypes.c_size_t]
class calls:
    start = staticmethod(shim.calls_start)
    refuse = staticmethod(shim.calls_refuse)
    stop = staticmethod(lambda: shim.calls_stop().decode())
arg = json.loads(sys.argv[2])
import numpy as np
from gpu_cases import Case
"""


def run(tmp_path, snippet, arg=None, timeout=100):
    """The JSON value the snippet passes to print(), its last line of output."""
    src, lib = tmp_path / "calls.c", tmp_path / "libcalls.so"
    src.write_text(SHIM)
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", str(lib), str(src), "-ldl"], check=True)
    env = dict(os.environ, PYTHONPATH=os.pathsep.join([ROOT, os.path.join(ROOT, "tests")]))
    r = subprocess.run([sys.executable, "-c", PRELUDE + snippet, str(lib), json.dumps(arg)], env=env, timeout=timeout,
                       capture_output=True, text=True)
    print(r.stdout[-2000:], r.stderr[-2000:], flush=True)
    assert r.returncode == 0
    return json.loads(r.stdout.strip().splitlines()[-1])
