"""x0 whose squares leave the range of the type (needs a GPU). Single solves: every compact form ends as
the standard form does, with its status, iterations and u(0) bit for bit, since it hands over to
it. Batches: NaN residuals of one instance end the call with ENUMERIC in both forms, and the next
call is not touched by it."""
import numpy as np
import pytest

import test_gpu_compact as TC
from paper_2103_14990_amd import dlmpc
from paper_2103_14990_amd import workloads as W

pytestmark = pytest.mark.gpu


def _end(p, x):
    try:
        r = p.solve(x, want_phi=True)
        return r.status, r.stats["iters"], r.stats["r_primal"], r.stats["r_dual"], r.u0.tobytes(), r.phi.tobytes()
    except dlmpc.DlmpcError as e:
        return (e.status,)


@pytest.mark.parametrize("precision,scales", [("fp64", (1e152, 1e154, 1e170, 1e300)), ("fp32", (1e17, 1e19, 1e25, 1e37))])
@pytest.mark.parametrize("mode", [TC.WHOLE, TC.INPUTS, TC.BLOCK])
def test_single_solves_end_as_the_standard_form(tmp_path, monkeypatch, precision, scales, mode):
    wl = W.workload("chain10")
    make = lambda **kw: dlmpc.Problem.from_network(wl.net, wl.d, wl.T, wl.cost, rho=5.0, eps=1e-4, max_iter=60,
                                                   precision=precision, **kw)
    p, g = TC._forced(tmp_path, monkeypatch, mode, make), make(schedule="graph")
    base = wl.x0(3)
    one = base.copy()
    one[7] *= scales[-1]
    for x in [base * s for s in scales[1:]] + [one]:
        assert _end(p, x) == _end(g, x)
    # in range still, the last power of ten: the compact form itself, up to rounding
    a, b = p.solve(base * scales[0]), g.solve(base * scales[0])
    assert a.status == b.status and a.stats["iters"] == b.stats["iters"]
    assert a.stats["schedule"] == (mode == TC.BLOCK)
    good = p.solve(base)
    ref = g.solve(base)
    assert good.stats["iters"] == ref.stats["iters"]
    assert TC.rel(good.u0, ref.u0) < (1e-9 if precision == "fp64" else 1e-4)
    p.close()
    g.close()


@pytest.mark.parametrize("rows,T", [(8, 10), (20, 15)])  # both recursions in one block, and two kernels
def test_batch_with_one_instance_out_of_range(rows, T):
    net = W.grid(rows, rows)
    p = dlmpc.Problem.from_network(net, 2, T, W.unit_cost(net), rho=5.0, eps=1e-3, max_iter=40, precision="fp32",
                                   max_batch=9, tune=False)
    assert p.info["batch_global"] == 1
    x = np.stack([W.x0(net, i) for i in range(9)])
    _, u, st = p.solve_batch(x)
    for scale in (1e20, 1e37):
        y = x.copy()
        y[4] *= scale
        with pytest.raises(dlmpc.DlmpcError) as e:
            p.solve_batch(y)
        assert e.value.status == dlmpc.ENUMERIC
        _, u2, st2 = p.solve_batch(x)
        assert np.array_equal(u, u2) and [q["iters"] for q in st] == [q["iters"] for q in st2]
    p.close()
