"""Single-instance solves in the compact form (needs a GPU): whole bases, input rows between the
plant's global recursions, and a whole solve in one workgroup, each forced through the tuning cache
and compared with the FP64 oracle after the same number of iterations.

Bars, as for the standard form: FP64 - equal counts, u(0), Phi and objective within 1e-9 relative;
FP32 - u(0) within 1e-4, objective within 1e-5. Sizes sit at the edges of the kernels: stops at each
of the first iterations (the form's cold start differs in the first three), one to four states,
several inputs, two time steps, more rows than a workgroup's lanes, patches with more rows than
the registers hold, state rows with more entries than they hold, one, two and four state rows per
thread, subsystems whose whole neighbourhood starts at zero."""
import functools

import numpy as np
import pytest

from oracle import dlmpc_oracle as O
from paper_2103_14990_amd import dlmpc
from paper_2103_14990_amd import workloads as W

pytestmark = pytest.mark.gpu

RHO = 5.0
WHOLE, INPUTS, BLOCK = 1, 2, 3


def rel(a, b):
    return float(np.abs(np.asarray(a) - np.asarray(b)).max() / max(np.abs(np.asarray(b)).max(), 1e-300))


def _net(kind, arg):
    if kind == "chain":
        return W.chain(arg)
    if kind == "paper":
        return W.paper_chain(arg)
    if kind == "grid":
        return W.grid(*arg)
    if kind == "star":
        return W.swing_network(f"star{arg}", arg, np.array([[0, i] for i in range(1, arg)]), 0)
    n, nx, nu, scale = arg
    return W.generic_network(n, W.chain_edges(n), nx, nu, 3, scale)


@functools.lru_cache(maxsize=2)
def _oracle(kind, arg, d, T, box):
    """Network, cost, and the oracle's iterates of a case (dense matrices: cases of both precisions share)."""
    net = _net(kind, arg)
    cost = W.paper_cost(net) if kind == "paper" else (W.box_cost(net) if box else W.unit_cost(net))
    try:
        pb = O.setup_from_network(net, d, T, cost)
    except Exception as e:  # locality that this plant does not allow
        pytest.skip(str(e))
    x0 = W.x0(net, 500, 0.2 if box and kind != "paper" else 1.0)
    hole = x0.copy()
    hole[: len(hole) // 2] = 0.0
    stops = [(1, x0), (2, x0), (3, x0), (4, x0), (25, x0), (7, hole), (5, 0 * x0)]
    if len(x0) > 1024:
        stops = [(4, hole)]
    return net, cost, [(n, x, O.solve(pb, x, RHO, 1e-14, n)) for n, x in stops]


def _forced(tmp_path, monkeypatch, mode, make):
    """The problem with the given form of single solves."""
    cache = tmp_path / "tune.txt"
    if not cache.exists():
        monkeypatch.setenv("DLMPC_TUNE_CACHE", str(cache))
        make().close()
    sig = cache.read_text().split("|")[0]
    cache.write_text(f"{sig}|phi_ntw=1 psi_capx=8 sched=0 glob=0 comp={mode}\n")
    monkeypatch.setenv("DLMPC_TUNE_CACHE", str(cache))
    p = make()
    monkeypatch.delenv("DLMPC_TUNE_CACHE")
    assert p.info["tune_cached"] == 1
    assert p.info["schedule"] == (mode == BLOCK) and p.info["psi_structured"] == (mode == INPUTS)
    return p


@pytest.mark.parametrize("kind,arg,d,T,box,precision,modes", [
    ("chain", 10, 1, 5, False, "fp64", (WHOLE, INPUTS, BLOCK)),
    ("chain", 10, 1, 5, False, "fp32", (WHOLE, INPUTS, BLOCK)),
    ("grid", (5, 7), 2, 6, True, "fp64", (WHOLE, INPUTS)),
    ("grid", (8, 8), 2, 10, False, "fp32", (WHOLE, INPUTS)),
    ("star", 40, 1, 5, False, "fp64", (WHOLE, INPUTS)),            # a hub of degree 39, 560-row patches
    ("paper", 12, 2, 10, True, "fp64", (WHOLE, INPUTS)),           # two inputs
    ("chain", 6, 1, 2, False, "fp64", (WHOLE, INPUTS, BLOCK)),     # two time steps
    ("generic", (9, 1, 1, 0.1), 1, 7, False, "fp64", (WHOLE, INPUTS, BLOCK)),
    ("generic", (9, 3, 3, 0.05), 1, 5, False, "fp64", (WHOLE, INPUTS)),
    ("generic", (7, 4, 4, 0.05), 1, 4, False, "fp64", (WHOLE, INPUTS)),
    ("chain", 3, 1, 180, False, "fp64", (WHOLE,)),                 # 539 rows per subsystem
    ("grid", (24, 24), 1, 3, True, "fp64", (WHOLE, INPUTS)),       # 1152 and 2080 states
    ("chain", 1040, 1, 2, True, "fp32", (WHOLE, INPUTS)),
    ("chain", 1040, 1, 2, True, "fp64", (INPUTS,)),
])
def test_compact_forms_match_oracle(tmp_path, monkeypatch, kind, arg, d, T, box, precision, modes):
    net, cost, refs = _oracle(kind, arg, d, T, box)
    f64 = precision == "fp64"
    for mode in modes:
        for iters, x, ref in refs:
            p = _forced(tmp_path, monkeypatch, mode, lambda: dlmpc.Problem.from_network(
                net, d, T, cost, rho=RHO, precision=precision, eps=1e-14, max_iter=iters))
            res = p.solve(x, want_phi=True)
            rp, ci = p.phi_pattern()
            phi = ref.Phi[np.repeat(np.arange(len(rp) - 1), np.diff(rp)), ci]
            eu, ep = rel(res.u0, ref.u0) if np.any(ref.u0) else float(np.abs(res.u0).max()), rel(res.phi, phi)
            print(f"  {net.name} {precision} mode {mode} iters {iters}: u0 rel {eu:.2e} phi rel {ep:.2e}", flush=True)
            # (from x0 = 0 every residual is the rounding of the offsets: which iteration sees it below
            # 1e-14 first is not determined, the fixed point is)
            assert res.stats["iters"] == ref.iters or not np.any(x)
            assert eu < (1e-9 if f64 else 1e-4) and ep < (1e-9 if f64 else 1e-4)
            assert abs(res.stats["objective"] - ref.J) <= (1e-9 if f64 else 1e-5) * ref.J + 1e-300
            for f, r in (("r_primal", ref.r_primal), ("r_dual", ref.r_dual)):
                assert abs(res.stats[f] - r) <= (1e-6 * r + 1e-9 if f64 else 1e-3 * r + 1e-6), f
            p.close()


@pytest.mark.parametrize("mode", [WHOLE, INPUTS, BLOCK])
def test_compact_state_after_the_stop(tmp_path, monkeypatch, mode):
    """The stop at eps, Psi and Lambda of the stopping iterate (through the certificate) and
    solves from a given start, which the standard form runs, against the graph schedule."""
    wl = W.workload("chain10")
    make = lambda **kw: dlmpc.Problem.from_network(wl.net, wl.d, wl.T, wl.cost, rho=RHO, eps=1e-4, max_iter=500, **kw)
    p, g = _forced(tmp_path, monkeypatch, mode, make), make(schedule="graph")
    for seed in (1, 2):
        a, b = p.solve(wl.x0(seed), want_phi=True), g.solve(wl.x0(seed), want_phi=True)
        assert a.stats["iters"] == b.stats["iters"] and a.status == b.status
        assert rel(a.u0, b.u0) < 1e-9 and rel(a.phi, b.phi) < 1e-9
        ca, cb = p.certify(), g.certify()
        for k in ca:
            assert abs(ca[k] - cb[k]) <= 1e-8 * max(1.0, abs(cb[k])), k
        zero = np.zeros(p.nnz)
        a, b = p.solve(wl.x0(seed), b.phi, zero), g.solve(wl.x0(seed), b.phi, zero)
        assert a.stats["iters"] == b.stats["iters"] and a.stats["schedule"] == 0
        assert rel(a.u0, b.u0) < 1e-9
    p.close()
    g.close()
