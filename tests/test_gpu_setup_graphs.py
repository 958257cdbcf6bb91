"""What a tuned setup of single solves captures and runs (needs a GPU). hipGraphInstantiate and
hipGraphLaunch are counted by a small library loaded ahead of the HIP runtime in a process of its own.

Each form that is timed needs one graph (the standard form with either Psi-comp, the compact form with
whole bases and through the global recursions), launched once to warm up and for up to three
samples; each form that is kept its set of six: at most 4 + 2 * 6 graphs, and 16 launches."""
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
long shim_graphs, shim_launches;
int hipGraphInstantiate(void **e, void *g, void *n, char *l, size_t s) {
  ++shim_graphs;
  return ((int (*)(void **, void *, void *, char *, size_t))real("hipGraphInstantiate"))(e, g, n, l, s);
}
int hipGraphLaunch(void *e, void *s) {
  ++shim_launches;
  return ((int (*)(void *, void *))real("hipGraphLaunch"))(e, s);
}
"""

CHILD = r"""
import ctypes as C, json, sys
shim = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)  # ahead of the HIP runtime
graphs, launches = C.c_long.in_dll(shim, "shim_graphs"), C.c_long.in_dll(shim, "shim_launches")
sys.path.insert(0, sys.argv[2])
from paper_2103_14990_amd import dlmpc
from paper_2103_14990_amd import workloads as W
net = W.paper_chain(40)
p = dlmpc.Problem.from_network(net, 2, 10, W.paper_cost(net), rho=5.0, precision="fp64", eps=1e-4, max_iter=500)
print(json.dumps(dict(graphs=graphs.value, launches=launches.value, tuned=p.info["tune_graph_us"])), flush=True)
p.close()
"""


def test_tuned_setup_captures_each_form_once(tmp_path):
    src, so = tmp_path / "shim.c", tmp_path / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", str(src), "-o", str(so), "-ldl"], check=True)
    env = {k: v for k, v in os.environ.items() if k != "DLMPC_TUNE_CACHE"}
    r = subprocess.run([sys.executable, "-u", "-c", CHILD, str(so), ROOT], capture_output=True, text=True, timeout=100, env=env)
    print(r.stdout[-2000:], r.stderr[-2000:], flush=True)
    assert r.returncode == 0
    n = json.loads([l for l in r.stdout.splitlines() if l.startswith("{")][0])
    assert n["tuned"] > 0
    assert 6 < n["graphs"] <= 16 and 4 < n["launches"] <= 16
