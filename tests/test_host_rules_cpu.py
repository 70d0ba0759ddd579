"""The host's rules for choosing among launches (csrc/host_rules.hpp), compiled
for the host alone and evaluated over their ranges."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_22684_amd", "csrc")


def evaluate(tmp_path, exprs):
    """Values of C++ expressions over namespace zk::rules."""
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("needs g++")
    src = tmp_path / "rules.cpp"
    body = "\n".join(f'  printf("%.17g\\n", (double)({e}));' for e in exprs)
    src.write_text(f'#include "host_rules.hpp"\n#include <cstdio>\nusing namespace zk::rules;\nint main() {{\n{body}\n}}\n')
    exe = str(tmp_path / "rules")
    subprocess.run([gxx, "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", exe], check=True)
    return [float(v) for v in subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()]


def test_msm_runs_are_never_a_long_serial_chain(tmp_path):
    """At every window size and number of points a lane may be asked for no
    fewer than 8 and no more than 32 entries when lanes are to spare, and for an
    eighth of an average bucket where that lies between."""
    cases = [(c, n) for c in range(1, 17) for n in (1, 50, 127, 511, 1000, 4096, 50000, 1 << 16, 1 << 20, 1 << 24)
             if -(-255 // c) * n < 1 << 32]
    got = evaluate(tmp_path, [f"msm_min_run({-(-255 // c)}, {n}ull, {c})" for c, n in cases])
    for (c, n), run in zip(cases, got):
        eighth = (-(-255 // c) * n) >> (c + 3)
        assert run == min(32, max(8, eighth)), f"c {c}, n {n}"
