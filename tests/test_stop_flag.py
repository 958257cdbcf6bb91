"""Kernels in which some blocks take the stop decision while others work: no working block may read
the flag that the same launch sets, wave by wave, ahead of a barrier (its waves could part there)."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2103_14990_amd", "csrc")


def _kernels(name):
    """Name and body of every kernel of a source file."""
    src = open(os.path.join(CSRC, name)).read()
    out = {}
    for m in re.finditer(r"__global__[^{;]*?\b(\w+)\((?:[^()]|\([^()]*\))*\) \{", src):
        out[m.group(1)] = src[m.end():src.index("\n}", m.end())]
    return out


def test_compact_kernels_that_decide_go_by_the_published_flag():
    ks = _kernels("single_compact.h")
    deciding = [n for n, b in ks.items() if "(a, c, true)" in b]
    assert sorted(deciding) == ["crow_kernel", "csim_fwd_kernel"]
    for n in deciding:
        assert "ctl->stop" not in ks[n] and "if (a.ctl->c_halt) return;" in ks[n], n
    # the flag's writers do not read it
    for n, b in ks.items():
        if re.search(r"c_halt = ", b):
            assert not re.search(r"if \([^)]*c_halt", b), n


def test_gather_blocks_read_the_flag_once():
    body = _kernels("batch_global.h")["bgather_kernel"]
    work = body[body.index("if (int(blockIdx.x) < N)"):body.index("a.init_pass")]
    assert work.count("ctl->stop") == 1 and "if (tid == 0) s_stop = a.ctl->stop;" in work
    assert "ctl->stop" not in body[:body.index("if (int(blockIdx.x) < N)")]
