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


def test_tiny_transforms_in_numbers_run_as_one_launch(tmp_path):
    """64 transforms of up to 2^6 points, an item each (two workgroups on each of
    256 CUs) are estimated, and measured, shorter as one launch; two of them are
    left to the persistent kernel.  A matrix-core pass has its floor."""
    sizes = range(2, 7)
    group = evaluate(tmp_path, [f"grouped_pass_us({k}, true, {jobs}, 256)" for jobs in (64, 2) for k in sizes])
    both = evaluate(tmp_path, ["persistent_us(64, 512)", "persistent_us(2, 512)"])
    assert all(t < both[0] for t in group[:5])
    assert all(t > both[1] for t in group[5:])
    floor, full = evaluate(tmp_path, ["grouped_pass_us(12, false, 1, 256)", "grouped_pass_us(18, false, 16, 256)"])
    assert floor == 10.0 and full == 4.0 + 4 * 33.0


def test_side_streams_by_the_way_a_batch_is_launched(tmp_path):
    """A graph's branches are free; without a graph each stream is paid for at
    every launch."""
    assert evaluate(tmp_path, ["side_streams(true)", "side_streams(false)"]) == [4, 3]


def test_whole_transforms_of_the_register_kernels(tmp_path):
    """Up to 2^7 points always, 2^8 to 2^10 in launches that fill the chip, 2^11
    never."""
    cases = [(0, 1, 1), (7, 1 << 7, 1), (7, 1 << 22, 1), (8, 1 << 8, 0), (8, (1 << 21) - (1 << 8), 0), (8, 1 << 21, 1),
             (9, 1 << 20, 0), (9, 1 << 21, 1), (10, 1 << 19, 0), (10, 1 << 20, 1), (11, 1 << 24, 0)]
    got = evaluate(tmp_path, [f"register_whole({n}, {e}ull)" for n, e, _ in cases])
    assert got == [c[2] for c in cases]
