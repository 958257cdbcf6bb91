"""Where the stop falls in a chunk of captured iterations (needs a GPU): after any number of iterations,
at the end of a chunk, inside it and in a later one, and solve after solve, a compact solve ends in
the same iterate bit for bit, and a batch likewise whatever its other instances do."""
import numpy as np
import pytest

import test_gpu_compact as TC
from paper_2103_14990_amd import dlmpc
from paper_2103_14990_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [TC.WHOLE, TC.INPUTS])
def test_compact_stop_anywhere_in_a_chunk(tmp_path, monkeypatch, mode):
    net = W.grid(5, 7)
    ref = {}
    for every in (32, 1, 2, 3, 7):
        p = TC._forced(tmp_path, monkeypatch, mode, lambda: dlmpc.Problem.from_network(
            net, 2, 6, W.box_cost(net), rho=5.0, precision="fp64", eps=1e-3, max_iter=200, check_every=every))
        for rep in range(2):
            for seed in range(4):
                r = p.solve(W.x0(net, 40 + seed, 0.1 + 0.1 * seed), want_phi=True)
                got = (r.stats["iters"], r.u0.tobytes(), r.phi.tobytes(), r.stats["r_primal"], r.stats["r_dual"])
                assert ref.setdefault(seed, got) == got, (every, rep, seed)
                # (the last x0 violates the box for good: its stop is that of max_iter)
                assert r.stats["converged"] == (seed < 3)
        p.close()
    assert len({v[0] for v in ref.values()}) > 1  # stops at different places


@pytest.mark.parametrize("rows", [6, 20])  # both recursions in one block, and two kernels
def test_batch_stop_does_not_depend_on_the_others(rows):
    net = W.grid(rows, rows)
    x = np.stack([W.x0(net, 60 + i, 0.05 + 0.02 * i) for i in range(9)])
    ref = {}
    for every in (32, 1, 5):
        p = dlmpc.Problem.from_network(net, 2, 15 if rows == 20 else 6, W.box_cost(net), rho=5.0, precision="fp32",
                                       eps=1e-3, max_iter=300, max_batch=9, tune=False, check_every=every)
        assert p.info["batch_global"] == 1
        for sel in (list(range(9)), [8, 0], [4]):
            _, u, st = p.solve_batch(x[sel])
            for q, i in enumerate(sel):
                got = (st[q]["iters"], u[q].tobytes(), st[q]["r_primal"], st[q]["r_dual"])
                assert ref.setdefault(i, got) == got, (every, sel, i)
        p.close()
    assert len({v[0] for v in ref.values()}) > 1
