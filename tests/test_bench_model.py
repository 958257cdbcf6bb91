"""bench.py's names and bytes of the batched engine's timed steps against what the library launches in
them (launch_one), for both ways of running the global recursions."""
import os
import re

import bench
from paper_2103_14990_amd import workloads as W

CSRC = os.path.join(os.path.dirname(os.path.abspath(bench.__file__)), "paper_2103_14990_amd", "csrc")
INFO = {"sum_dcol_k": 1000, "sum_k": 70, "n_tiles": 30, "sum_du_k": 400, "batch_global": 1, "input_rows": 4}


def test_fused_sizes_are_the_library_s():
    src = open(os.path.join(CSRC, "batch_kernels.hip")).read()
    m = re.search(r"sim_both_ = N <= kSimThreads && sim_rpt\(\) <= 2 && size_t\(N\) \* hs.rs \* sizeof\(float\) <= kSimBothLds;", src)
    assert m and re.search(r"kSimBothLds = 64 \* 1024;", src)
    assert re.search(r"kSimThreads = 1024;", open(os.path.join(CSRC, "batch_global.h")).read())
    assert bench.recursions_fused(1024, 2, 16) and not bench.recursions_fused(1024, 2, 17)
    assert not bench.recursions_fused(1025, 1, 2) and not bench.recursions_fused(1024, 3, 4)
    wl = W.workload("irregular1024_box")
    assert not bench.recursions_fused(wl.net.n_sub, wl.net.nx, wl.net.nx * wl.T + wl.net.nu * (wl.T - 1))


def test_steps_and_bytes():
    N, rs, B = 5, 14, 3
    two = bench.batch_algorithmic_bytes({**INFO, "recursions_fused": False}, N, rs, B)
    one = bench.batch_algorithmic_bytes({**INFO, "recursions_fused": True}, N, rs, B)
    g, alpha = 4 * B * N * 4, 4 * B * N * rs
    assert one["bphi_kernel"] == two["bphi_kernel"] + g            # g is written by the first step
    assert one["bpsi_kernel"] == two["bpsi_kernel"] - g - alpha    # and alpha is not read again
    assert one["bdecide_kernel"] == two["bdecide_kernel"]
    assert bench.FUSED_KERNELS["bphi_kernel"] == "bsim_both_kernel" and bench.FUSED_KERNELS["bpsi_kernel"] == "bstep_kernel"
    for k in "bsim_fwd_kernel bsim_adj_kernel bsim_both_kernel bstep_kernel bgather_kernel".split():
        assert len(bench.kernel_source_hash(k)) == 16
