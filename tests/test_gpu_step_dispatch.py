"""Every instance of bstep_kernel that a launch can pick (needs a GPU): one to four tiles of basis
vectors per wave (null-space dimensions up to 128, 256, 384 and 512), 16 and 32 instances per block,
chosen by max_batch and by the LDS that 32 instances of a patch need, with remainders of instances
and basis vectors. Compared with FP64 single solves of the standard form after the same number of
iterations; bars of the FP32 tier (u(0) 1e-4, objective 1e-5)."""
import numpy as np
import pytest

from paper_2103_14990_amd import dlmpc
from paper_2103_14990_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,arg,d,T,B,max_batch,tiles", [
    ("grid", (6, 6), 2, 9, 5, 5, 1),
    ("paper", 16, 2, 12, 18, 20, 1),      # k_max 100: one tile per wave, all eight waves, 32 instances
    ("grid", (6, 6), 3, 9, 5, 16, 2),     # k_max 136
    ("grid", (6, 6), 3, 9, 18, 33, 2),
    ("mesh", (8, 8), 3, 15, 3, 3, 3),     # k_max 258
    ("mesh", (8, 8), 3, 15, 17, 20, 3),
    ("mesh", (8, 8), 4, 12, 33, 40, 3),   # k_max 368
    ("grid", (7, 7), 4, 15, 4, 16, 4),    # k_max 422
    ("grid", (7, 7), 4, 15, 33, 40, 4),
    ("grid", (8, 8), 4, 15, 20, 64, 4),   # k_max 402; 32 instances of a patch of 39 do not fit twice on a CU
])
def test_batch_matches_fp64_single_solves(kind, arg, d, T, B, max_batch, tiles):
    net = W.grid(*arg) if kind == "grid" else (W.paper_chain(arg) if kind == "paper" else W.irregular_mesh(*arg, 0))
    cost = W.paper_cost(net) if kind == "paper" else W.box_cost(net)
    make = lambda **kw: dlmpc.Problem.from_network(net, d, T, cost, rho=5.0, eps=1e-14, max_iter=20, **kw)
    p, ref = make(precision="fp32", max_batch=max_batch, tune=False), make(precision="fp64", schedule="graph")
    assert p.info["batch_global"] == 1 and (p.info["k_max"] + 127) // 128 == tiles
    x0 = np.stack([W.x0(net, 300 + i, 1.0 if kind == "paper" else 0.2) for i in range(B)])
    _, u, st = p.solve_batch(x0)
    for i in sorted({0, B // 2, B - 1}):
        r = ref.solve(x0[i])
        e = float(np.abs(u[i] - r.u0).max() / np.abs(r.u0).max())
        print(f"  {net.name} d {d} T {T} k_max {p.info['k_max']} instance {i}: u0 rel {e:.2e}", flush=True)
        assert st[i]["iters"] == r.stats["iters"] == 20
        assert e < 1e-4 and abs(st[i]["objective"] - r.stats["objective"]) <= 1e-5 * r.stats["objective"]
    p.close()
    ref.close()
