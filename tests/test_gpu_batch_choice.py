"""How setup chooses between the dense products and the global recursions of the batched engine (needs
a GPU): by captured iterations, as solves run them, not by launches timed one by one.

hipGraphLaunch and the kernel nodes of its graphs are counted by a small library loaded ahead of the
HIP runtime in a process of its own: each form is launched once to warm up and for up to three
samples of as many iterations, three kernels each on a network whose recursions run in one kernel."""
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
static void *real(const char *name) {
  void *h = dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD);
  if (!h) h = dlopen("libamdhip64.so", RTLD_LAZY | RTLD_NOLOAD);
  return h ? dlsym(h, name) : NULL;
}
long shim_launches, shim_nodes[64];
static struct { void *exec; size_t nodes; } tab[256];
int hipGraphInstantiate(void **e, void *g, void *n, char *l, size_t s) {
  size_t nodes = 0;
  ((int (*)(void *, void **, size_t *))real("hipGraphGetNodes"))(g, NULL, &nodes);
  int rc = ((int (*)(void **, void *, void *, char *, size_t))real("hipGraphInstantiate"))(e, g, n, l, s);
  for (int i = 0; i < 256; ++i)
    if (!tab[i].exec || tab[i].exec == *e) { tab[i].exec = *e; tab[i].nodes = nodes; break; }
  return rc;
}
int hipGraphLaunch(void *e, void *s) {
  for (int i = 0; i < 256; ++i)
    if (tab[i].exec == e && shim_launches < 64) shim_nodes[shim_launches] = (long)tab[i].nodes;
  ++shim_launches;
  return ((int (*)(void *, void *))real("hipGraphLaunch"))(e, s);
}
"""

CHILD = r"""
import ctypes as C, json, sys
shim = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)  # ahead of the HIP runtime
n, nodes = C.c_long.in_dll(shim, "shim_launches"), (C.c_long * 64).in_dll(shim, "shim_nodes")
sys.path.insert(0, sys.argv[2])
from paper_2103_14990_amd import dlmpc
from paper_2103_14990_amd import workloads as W
net = W.paper_chain(22)
p = dlmpc.Problem.from_network(net, 1, 6, W.paper_cost(net), rho=5.0, precision="fp32", eps=1e-3, max_iter=100, max_batch=4,
                               schedule="graph")
print(json.dumps(dict(nodes=list(nodes[:n.value]))), flush=True)
p.close()
"""


def test_both_forms_are_timed_as_captured_iterations(tmp_path):
    src, so = tmp_path / "shim.c", tmp_path / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", str(src), "-o", str(so), "-ldl"], check=True)
    env = {k: v for k, v in os.environ.items() if k != "DLMPC_TUNE_CACHE"}
    r = subprocess.run([sys.executable, "-u", "-c", CHILD, str(so), ROOT], capture_output=True, text=True, timeout=100, env=env)
    print(r.stdout[-2000:], r.stderr[-2000:], flush=True)
    assert r.returncode == 0
    nodes = json.loads([l for l in r.stdout.splitlines() if l.startswith("{")][0])["nodes"]
    assert 4 <= len(nodes) <= 8 and nodes[0] == 3 * 8
    assert len(set(nodes)) == 1  # phi, psi, decide; both recursions, step, gather
