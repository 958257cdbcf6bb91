"""Setup when device memory runs out (needs a GPU). hipMalloc is interposed by a small library loaded
ahead of the HIP runtime in a process of its own; it counts the calls and the bytes held, and
answers a chosen call, or what would pass a chosen total, with out-of-memory.

The iteration through the global recursions and the compact form of single solves are optional: a
failed allocation of theirs leaves setup on the other form, holding what it would have held without
the attempt, and they come after every allocation that setup cannot do without."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>
typedef int (*malloc_t)(void **, size_t);
typedef int (*free_t)(void *);
static void *real(const char *name) {
  void *h = dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD);
  if (!h) h = dlopen("libamdhip64.so", RTLD_LAZY | RTLD_NOLOAD);
  return h ? dlsym(h, name) : NULL;
}
enum { MAX = 1 << 16 };
static void *ptr[MAX];
static size_t size[MAX];
static long calls, first, last;
static size_t live;
void shim_arm(long f, long l) { calls = 0; first = f; last = l; }
long shim_calls(void) { return calls; }
size_t shim_live(void) { return live; }
int hipMalloc(void **p, size_t n) {
  static malloc_t f;
  if (!f) f = (malloc_t)real("hipMalloc");
  ++calls;
  if (calls >= first && calls <= last) return 2; /* hipErrorOutOfMemory */
  int rc = f(p, n);
  for (int i = 0; rc == 0 && i < MAX; ++i)
    if (!ptr[i]) { ptr[i] = *p; size[i] = n; live += n; break; }
  return rc;
}
int hipFree(void *p) {
  static free_t f;
  if (!f) f = (free_t)real("hipFree");
  for (int i = 0; p && i < MAX; ++i)
    if (ptr[i] == p) { ptr[i] = NULL; live -= size[i]; break; }
  return f(p);
}
"""

CHILD = r"""
import ctypes as C, json, sys
shim = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)  # ahead of the HIP runtime
shim.shim_arm.argtypes = [C.c_long, C.c_long]
shim.shim_calls.restype = C.c_long
shim.shim_live.restype = C.c_size_t
sys.path.insert(0, sys.argv[2])
import numpy as np
from paper_2103_14990_amd import dlmpc
from paper_2103_14990_amd import workloads as W
wl = W.workload("grid8" if sys.argv[3] == "batch" else "chain10")
x0 = np.stack([wl.x0(s) for s in range(3)])
NONE = (0, -1)

def make():
    if sys.argv[3] == "batch":
        return dlmpc.Problem.from_network(wl.net, wl.d, wl.T, wl.cost, rho=5.0, precision="fp32", eps=1e-3, max_iter=500,
                                          max_batch=5, tune=False, schedule="graph")
    return dlmpc.Problem.from_network(wl.net, wl.d, wl.T, wl.cost, rho=5.0, precision="fp64", eps=1e-4, max_iter=500)

def solve(p):
    return p.solve_batch(x0)[1] if sys.argv[3] == "batch" else np.stack([p.solve(x).u0 for x in x0])

make().close()  # the runtime's own allocations
base = shim.shim_live()

def attempt(first, last):
    shim.shim_arm(first, last)
    try:
        p = make()
    except dlmpc.DlmpcError as e:
        out = dict(status=e.status, live=shim.shim_live() - base, calls=shim.shim_calls())
        shim.shim_arm(*NONE)
        return out
    out = dict(status=0, live=shim.shim_live() - base, calls=shim.shim_calls(),
               glob=p.info["batch_global"])
    shim.shim_arm(*NONE)
    u = solve(p)
    out["err"] = float(np.abs(u - ref).max() / np.abs(ref).max())
    p.close()
    out["left"] = shim.shim_live() - base
    return out

p = make(); ref = solve(p); p.close()
full = attempt(*NONE)
print(json.dumps(dict(full=full)), flush=True)
for last in (0, 1 << 30):  # a single failed call; every call from the n-th on
    for n in range(1, full["calls"] + 1):
        print(json.dumps(dict(n=n, single=last == 0, **attempt(n, last or n))), flush=True)
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("shim")
    src, so = d / "shim.c", d / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", str(src), "-o", str(so), "-ldl"], check=True)
    return str(so)


def _run(shim, kind):
    env = {k: v for k, v in os.environ.items() if k != "DLMPC_TUNE_CACHE"}
    r = subprocess.run([sys.executable, "-u", "-c", CHILD, shim, ROOT, kind], capture_output=True, text=True, timeout=100,
                       env=env)
    print(r.stdout[-4000:], r.stderr[-2000:], flush=True)
    assert r.returncode == 0
    out = [json.loads(l) for l in r.stdout.splitlines() if l.startswith("{")]
    full, rows = out[0]["full"], out[1:]
    assert full["status"] == 0 and full["left"] == 0
    assert len(rows) == 2 * full["calls"] > 80 and rows[0]["status"]
    for r in rows:
        if r["status"]:
            assert r["live"] == 0  # a setup that fails gives everything back
        else:
            assert r["left"] == 0 and r["err"] < 1e-4
    return full, [[r for r in rows if r["single"] == q and r["status"] == 0] for q in (True, False)]


def test_batched_setup_without_memory_for_the_global_recursions(shim):
    full, (one, rest) = _run(shim, "batch")
    assert full["glob"] == 1
    # whichever of its allocations failed, and whatever is left for those after it, setup ends with the
    # dense products and holds the same
    assert len(one) > 10 and [r["n"] for r in one] == [r["n"] for r in rest]
    assert all(r["glob"] == 0 for r in one + rest)
    assert len({r["live"] for r in one + rest}) == 1


def test_single_setup_without_memory_for_the_compact_form(shim):
    _, (_, rest) = _run(shim, "single")
    # every allocation of the compact form may fail; what is held is that of the forms that are left:
    # the standard one, and from the global recursions' buffers on, the whole bases' beside it
    live = [r["live"] for r in rest]
    assert len(live) > 20 and live == sorted(live) and len(set(live)) <= 2
