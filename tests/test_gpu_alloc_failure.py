"""Updates that run out of memory: every allocation that an update makes is made to
fail once, in a process of its own whose allocation calls go through a small library
that this test builds.  The update must report KATZ_E_OOM and leave the state as it
was: small updates and their inverses go on to certify the ranking that stood before,
and once no allocation fails the update gives what it gives elsewhere."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#define _GNU_SOURCE
#include <dlfcn.h>
#include <link.h>
#include <stddef.h>
#include <string.h>

static int countdown, calls;

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

static int fails(void) {
  ++calls;
  return countdown > 0 && --countdown == 0;
}

void arm(int nth) { countdown = nth; }
int seen(void) { return calls; }

int hipMalloc(void** p, size_t bytes) {
  static int (*f)(void**, size_t);
  if (!f) f = (int (*)(void**, size_t))real("hipMalloc");
  return fails() || !f ? 2 : f(p, bytes);
}

int hipHostMalloc(void** p, size_t bytes, unsigned flags) {
  static int (*f)(void**, size_t, unsigned);
  if (!f) f = (int (*)(void**, size_t, unsigned))real("hipHostMalloc");
  return fails() || !f ? 2 : f(p, bytes, flags);
}
"""

CHILD = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)   # before the HIP runtime: its names come first
directed = sys.argv[2] == "directed"
import numpy as np
import torch
import synthgraph as sg
import paper_1807_03847_amd.katz as katz

n = 4000
rng = np.random.default_rng(5)
rp, col = sg.rmat_directed(12, 8, seed=4) if directed else sg.barabasi_albert(n, 6, 9)
n = len(rp) - 1
src = np.repeat(np.arange(n), np.diff(rp))
arcs = set(zip(src.tolist(), np.asarray(col).tolist()))
cap = sg.max_degree(rp) + 20000
alpha, k = 0.5 / (1 + cap), 30
dev = lambda a, t: torch.from_numpy(np.ascontiguousarray(np.asarray(a, dtype=t))).cuda()
make = lambda rp, col: katz.create_state(dev(rp, np.int64), dev(col, np.int32), k, alpha=alpha, eps=1e-9,
                                         degree_cap=cap, undirected=not directed)
state, first = make(rp, col)
out = [torch.empty(k, dtype=t, device="cuda") for t in (torch.int32, torch.float64, torch.float64)]

def update(ins=None, dels=None, fail=0):
    shim.arm(fail)
    try:
        state.update(ins, dels, out=out)
    finally:
        shim.arm(0)
    return [t.clone() for t in out]

def absent(count, seed):
    g = np.random.default_rng(seed)
    found = set()
    while len(found) < count:
        a, b = (int(v) for v in g.integers(0, n, 2))
        if a != b and (a, b) not in arcs and (b, a) not in arcs and (b, a) not in found:
            found.add((a, b))
    return np.array(sorted(found), dtype=np.int32)

assert shim.seen() > 0, "the library's allocations do not pass the shim"
small = absent(3, 1)
update(small)
base = update(None, small)
big = np.array([p for p in absent(40000, 2).tolist() if tuple(p) not in set(map(tuple, small.tolist()))], dtype=np.int32)
failed = 0
for nth in range(1, 40):
    print("[gpu-case] allocation", nth, "directed" if directed else "undirected", flush=True)
    try:
        after = update(big, fail=nth)
    except katz.KatzError as e:
        assert e.code == katz.E_OOM, e
        failed += 1
        update(small)
        again = update(None, small)
        assert all(torch.equal(a, b) for a, b in zip(base, again)), nth
        continue
    break
else:
    raise SystemExit("the update never went through")
assert failed >= (8 if directed else 6), failed
both = big if directed else np.concatenate([big, big[:, ::-1]])
new = np.array(sorted(arcs | set(map(tuple, both.tolist()))), dtype=np.int64)
rp2, col2 = sg.from_edges(n, new[:, 0], new[:, 1], undirected=False)
r = state.update(out=out).iterations
lo, up = katz.bounds(dev(rp2, np.int64), dev(col2, np.int32), r, alpha=alpha, undirected=not directed)
ids = after[0].long()
assert torch.equal(lo[ids], after[1]) and torch.equal(up[ids], after[2])
state.free()
print("failed", failed, "ok")
"""


@pytest.mark.parametrize("form", ["undirected", "directed"])
def test_update_survives_every_failed_allocation(tmp_path, form):
    src = tmp_path / "shim.c"
    src.write_text(SHIM)
    lib = str(tmp_path / "libshim.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", str(src), "-o", lib, "-ldl"], check=True)
    env = dict(os.environ, PYTHONPATH=ROOT + os.pathsep + os.environ.get("PYTHONPATH", ""))
    run = subprocess.run([sys.executable, "-u", "-c", CHILD, lib, form], cwd=ROOT, env=env, capture_output=True,
                         text=True, timeout=110)
    print(run.stdout[-3000:], flush=True)
    assert run.returncode == 0, run.stdout[-1500:] + run.stderr[-3000:]
    assert run.stdout.rstrip().endswith("ok")
