"""A log of the kernels that the library launches, and on which streams, and of its waits
for streams: a small library, built with gcc, whose hipLaunchKernel and
hipStreamSynchronize come before the runtime's in a process that loads it first.  Used by tests that run a child process (``run_child``)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#define _GNU_SOURCE
#include <dlfcn.h>
#include <link.h>
#include <string.h>

typedef struct { unsigned x, y, z; } Dim;
enum { MAX = 1 << 16 };
static struct { const void* f; void* stream; } seen[MAX];
static int count;

static int find(struct dl_phdr_info* i, size_t n, void* out) {
  (void)n;
  if (!i->dlpi_name || !strstr(i->dlpi_name, "libamdhip64")) return 0;
  *(void**)out = dlopen(i->dlpi_name, RTLD_LAZY | RTLD_NOLOAD);
  return *(void**)out != NULL;
}

static void* real(const char* name) {
  static void* lib;
  if (!lib) dl_iterate_phdr(find, &lib);
  return lib ? dlsym(lib, name) : NULL;
}

int hipLaunchKernel(const void* f, Dim grid, Dim block, void** args, size_t lds, void* stream) {
  static int (*go)(const void*, Dim, Dim, void**, size_t, void*);
  if (!go) go = (int (*)(const void*, Dim, Dim, void**, size_t, void*))real("hipLaunchKernel");
  const int at = __atomic_fetch_add(&count, 1, __ATOMIC_RELAXED);
  if (at < MAX) {
    seen[at].f = f;
    seen[at].stream = stream;
  }
  return go(f, grid, block, args, lds, stream);
}

static int syncs;

int hipStreamSynchronize(void* stream) {
  static int (*go)(void*);
  if (!go) go = (int (*)(void*))real("hipStreamSynchronize");
  __atomic_fetch_add(&syncs, 1, __ATOMIC_RELAXED);
  return go(stream);
}

void log_clear(void) { count = syncs = 0; }
int log_syncs(void) { return syncs; }
int log_count(void) { return count < MAX ? count : MAX; }
void* log_stream(int i) { return seen[i].stream; }
const char* log_name(int i) {
  static const char* (*name)(const void*, void*);
  if (!name) name = (const char* (*)(const void*, void*))real("hipKernelNameRefByPtr");
  const char* n = name ? name(seen[i].f, NULL) : NULL;
  return n ? n : "?";
}
"""

PRELUDE = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)   # before the HIP runtime: its names come first
shim.log_name.restype = ctypes.c_char_p
shim.log_stream.restype = ctypes.c_void_p

def launches(call):
    "The library's launches in call(): (kernel name, stream handle) each."
    shim.log_clear()
    out = call()
    log = [(shim.log_name(i).decode(), shim.log_stream(i) or 0) for i in range(shim.log_count())]
    log = [(n, s) for n, s in log if "katz" in n]
    assert log, "the library's launches do not pass the log"
    return out, log

import numpy as np
import torch
import synthgraph as sg
import paper_1807_03847_amd.katz as katz
"""


def run_child(tmp_path, code, *args, timeout=110):
    """Runs PRELUDE and code in a child process; returns its output."""
    src = tmp_path / "launch_log.c"
    src.write_text(SHIM)
    lib = str(tmp_path / "liblaunch_log.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", str(src), "-o", lib, "-ldl"], check=True)
    env = dict(os.environ, PYTHONPATH=ROOT + os.pathsep + os.environ.get("PYTHONPATH", ""))
    run = subprocess.run([sys.executable, "-u", "-c", PRELUDE + code, lib, *args], cwd=ROOT, env=env,
                         capture_output=True, text=True, timeout=timeout)
    print(run.stdout[-3000:], flush=True)
    assert run.returncode == 0, run.stdout[-1500:] + run.stderr[-3000:]
    return run.stdout
