"""The FP64 certificate at the edges of its kernel's splits (needs a GPU): more rows per subsystem than
threads, fewer rows than groups, hubs, basis counts that are no multiple of eight, one to four
columns. Against the oracle's Phi and Psi after the same iterations: |Phi - Psi|, the primal
residual and the bound violation within 1e-9 of the largest entry; the feasibility and
stationarity residuals of an exact projection stay at rounding."""
import numpy as np
import pytest

from oracle import dlmpc_oracle as O
from paper_2103_14990_amd import dlmpc
from paper_2103_14990_amd import workloads as W

pytestmark = pytest.mark.gpu


def _star(n):
    return W.swing_network(f"star{n}", n, np.array([[0, i] for i in range(1, n)]), 0)


@pytest.mark.parametrize("make,d,T,box", [
    (lambda: W.chain(3), 1, 180, False),                                       # 539 rows per subsystem
    (lambda: W.chain(6), 1, 2, False),
    (lambda: _star(40), 1, 5, False),
    (lambda: W.grid(5, 7), 2, 6, True),
    (lambda: W.generic_network(9, W.chain_edges(9), 1, 1, 3, 0.1), 1, 7, False),
    (lambda: W.generic_network(7, W.chain_edges(7), 4, 4, 3, 0.05), 1, 4, False),
])
@pytest.mark.parametrize("iters", [1, 6])
def test_certificate_values(make, d, T, box, iters):
    net = make()
    cost = W.box_cost(net) if box else W.unit_cost(net)
    pb = O.setup_from_network(net, d, T, cost)
    x0 = W.x0(net, 77, 0.2 if box else 1.0)
    ref = O.solve(pb, x0, 5.0, 1e-14, iters)
    p = dlmpc.Problem.from_network(net, d, T, cost, rho=5.0, eps=1e-14, max_iter=iters, precision="fp64")
    p.solve(x0)
    c = p.certify()
    scale = max(1.0, float(np.abs(ref.Phi).max()))
    diff = ref.Phi - ref.Psi
    print(f"  {net.name} iters {iters}: {c}", flush=True)
    assert abs(c["pf"] - np.abs(diff).max()) < 1e-9 * scale
    assert abs(c["rp"] - np.sqrt((diff ** 2).sum(0)).max()) < 1e-9 * scale
    assert c["eq"] < 1e-9 * scale and c["stat"] < 1e-9 * scale * 5.0
    if not box:
        assert c["box"] == 0.0
    p.close()
