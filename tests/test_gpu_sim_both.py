"""Batched solves on either side of the line between one block per instance for both global
recursions and the two kernels (needs a GPU): 64 KB of rows per instance, 1024 subsystems, one or two
state rows per thread, subsystems that do not divide the block. Compared with FP64 single solves of
the standard form after the same number of iterations; bars of the FP32 tier (u(0) 1e-4, objective 1e-5)."""
import numpy as np
import pytest

from paper_2103_14990_amd import dlmpc
from paper_2103_14990_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,arg,d,T,box,B,max_batch", [
    ("grid", (19, 19), 2, 15, True, 5, 5),        # 15884 rows: one block, 361 subsystems
    ("grid", (20, 20), 2, 15, True, 5, 9),        # 17600 rows: two kernels
    ("chain", 1024, 1, 5, False, 3, 3),           # 14336 rows, 2048 states: one block, two rows per thread
    ("chain", 1025, 1, 5, False, 2, 3),           # 1025 subsystems: two kernels
    ("paper", 100, 2, 12, True, 33, 40),          # two inputs
    ("chain", 3, 1, 15, False, 2, 2),             # a few rows, 128 threads
])
def test_batch_matches_fp64_single_solves(kind, arg, d, T, box, B, max_batch):
    net = W.chain(arg) if kind == "chain" else (W.paper_chain(arg) if kind == "paper" else W.grid(*arg))
    cost = W.paper_cost(net) if kind == "paper" else (W.box_cost(net) if box else W.unit_cost(net))
    make = lambda **kw: dlmpc.Problem.from_network(net, d, T, cost, rho=5.0, eps=1e-14, max_iter=20, **kw)
    p, ref = make(precision="fp32", max_batch=max_batch, tune=False), make(precision="fp64", schedule="graph")
    assert p.info["batch_global"] == 1
    x0 = np.stack([W.x0(net, 900 + i, 0.2 if box and kind != "paper" else 1.0) for i in range(B)])
    _, u, st = p.solve_batch(x0)
    for i in {0, B // 2, B - 1}:
        r = ref.solve(x0[i])
        e = float(np.abs(u[i] - r.u0).max() / np.abs(r.u0).max())
        print(f"  {net.name} instance {i}: u0 rel {e:.2e}", flush=True)
        assert st[i]["iters"] == r.stats["iters"] == 20
        assert e < 1e-4 and abs(st[i]["objective"] - r.stats["objective"]) <= 1e-5 * r.stats["objective"]
    p.close()
    ref.close()
