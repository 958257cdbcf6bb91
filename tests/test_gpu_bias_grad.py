"""Bias gradients of the warm-start network, summed over the samples by the waves of a block (needs
a GPU): one sample, fewer samples than waves, an unrolled round with a remainder, and layer widths
of one, a full and a partial 64-column tile, against the FP64 reference network. Bar: that of the
other gradient blocks, 1e-4 relative (the layers above are split-bf16 products)."""
import numpy as np
import pytest

import test_gpu_warmstart as TW
from oracle import dlmpc_oracle as O
from oracle import mlp_ref as M
from paper_2103_14990_amd import dlmpc
from paper_2103_14990_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,H", [(1, 64), (7, 1), (16, 65), (127, 64), (128, 63), (129, 130), (300, 64)])
def test_bias_gradients(S, H):
    torch = pytest.importorskip("torch")
    wl = W.workload("chain10")
    pb = O.setup_from_network(wl.net, wl.d, wl.T, wl.cost)
    pr = dlmpc.Problem.from_network(wl.net, wl.d, wl.T, wl.cost, rho=5.0, precision="fp32", max_batch=4)
    pr.ws_init(H, S, seed=2, x_scale=0.8, y_scale=0.1)
    sh = pr.ws_shape()
    G, IN, OUT = wl.net.n_sub, sh["IN"], sh["OUT"]
    rng = np.random.default_rng(S + H)
    x0s, y = rng.standard_normal((S, G * wl.net.nx)), 0.1 * rng.standard_normal((S, G * TW.rows(wl)))
    xd, yd = torch.tensor(x0s, device="cuda"), torch.tensor(y, device="cuda")
    _, g = pr.ws_loss_grad(S, xd.data_ptr(), yd.data_ptr())
    Yt = (y / 0.1).reshape(S, G, -1)[:, :, wl.net.nx * wl.T:].transpose(1, 0, 2)
    theta = M.unflatten(pr.ws_params().astype(np.float64), G, IN, H, OUT)
    _, ref = M.loss_and_grads(theta, TW.network_inputs(pb, x0s, IN, 0.8), Yt)
    got = M.unflatten(g.astype(np.float64), G, IN, H, OUT)
    for q, name in ((1, "b1"), (3, "b2"), (5, "b3")):
        e = np.linalg.norm(got[q] - ref[q]) / np.linalg.norm(ref[q])
        print(f"  S {S} H {H} d{name}: rel {e:.2e}", flush=True)
        assert e < 1e-4
    pr.close()
