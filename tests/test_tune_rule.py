"""The autotuner's rule for a candidate against the form kept so far, and that every choice in the
library goes through it."""
import ctypes
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2103_14990_amd", "csrc")


@pytest.mark.parametrize("us,kept,want", [
    (98.9, 100.0, True), (50.0, 100.0, True),
    (99.0, 100.0, False), (99.5, 100.0, False), (100.0, 100.0, False), (120.0, 100.0, False),
    (0.0, 100.0, False),              # not timed
    (float("nan"), 100.0, False), (50.0, float("nan"), False),
])
def test_margin(tmp_path, us, kept, want):
    src, so = tmp_path / "rule.cpp", tmp_path / "rule.so"
    src.write_text('#include "tune_rule.h"\nextern "C" int rule(double a, double b) { return dlmpc::replaces(a, b); }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    f = ctypes.CDLL(str(so)).rule
    f.argtypes = [ctypes.c_double, ctypes.c_double]
    assert bool(f(us, kept)) == want


def test_every_choice_uses_the_rule():
    """Timings (tune_*_us, the sums of launches, a compact form's time) are compared by it alone."""
    src = open(os.path.join(CSRC, "dlmpc_api.cpp")).read()
    body = src[src.index("int tune_batch("):src.rindex("int setup_batch(")] + \
        src[src.index("int choose_schedule(dlmpc_problem *p) {"):src.index("bool finite_all(")]
    assert len(re.findall(r"dlmpc::replaces\(", body)) == 6
    assert not re.search(r"(tune_\w+_us(\[\w+\])?|\bsum|\bt) *[<>] *(0\.99|best_us|dense|p->tune)", body)
