"""When the spread gives each bin group of a patch of several rounds a work
item of its own (csrc/plan_sizes.hpp, spread_split), on the CPU: only where
the launch would end in a tail. The counts are those of random and of warped
sensor layouts; with the device filled many times over the finer items only
read the slots twice as often."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1510_01078_amd", "csrc")

# (patches, rounds over all of them, of the largest, bin groups) -> split
CASES = [
    ((576, 1160, 3, 18), True),      # 192^2 grid: 5184 items, barely one fill
    ((576, 1069, 9, 18), True),      # the same grid, a dense patch
    ((2304, 4637, 3, 34), False),    # 384^2 grid: 39168 items, 8 fills
    ((2304, 4171, 14, 34), False),   # the same grid warped: its longest item is an average share
    ((2304, 4171, 40, 34), True),    # one far denser patch
    ((1296, 2600, 3, 26), False),    # 288^2 grid: 16848 items
    ((1024, 1309, 2, 27), False),    # 256^2 grid: 14336 items
    ((1024, 2048, 3, 21), True),     # the same with a narrower band: 11264 items
    ((1, 1, 1, 1), True),
    ((1 << 24, 1 << 26, 1 << 20, 512), False),  # no overflow at the largest grids
]


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_spread_split(tmp_path):
    body = "\n".join(f'  std::printf("%d\\n", patsz::spread_split({p}LL, {r}LL, {m}LL, {c}) ? 1 : 0);'
                     for (p, r, m, c), _ in CASES)
    src = tmp_path / "split.cpp"
    src.write_text('#include <cstdio>\n#include "plan_sizes.hpp"\nint main() {\n' + body + "\n  return 0;\n}\n")
    exe = tmp_path / "split"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True,
                   capture_output=True, timeout=120)
    got = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout.split()
    assert [bool(int(v)) for v in got] == [w for _, w in CASES]
