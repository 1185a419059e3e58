"""How the backward pass cuts a sink block's column (csrc/pattern.h, compiled for the CPU): parts are short only where the
launch is small, whatever the window, and the launch stays inside the limits of a grid."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
POWER = 1

SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include "pattern.h"
int main(int argc, char** argv) {
  long long a[7];
  for (int i = 0; i < 7; ++i) a[i] = atoll(argv[i + 1]);
  printf("%d\n", pa_sink_part(a[0], (int32_t)a[1], (int32_t)a[2], (uint32_t)a[3], a[4], (int32_t)a[5], (int32_t)a[6]));
}
"""


@pytest.fixture(scope="module")
def part(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs a C++ compiler")
    d = tmp_path_factory.mktemp("part")
    (d / "part.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2503_03588_amd", "csrc"), str(d / "part.cpp"),
                    "-o", str(d / "part")], check=True, timeout=120)
    return lambda *a: int(subprocess.run([str(d / "part"), *map(str, a)], capture_output=True, text=True, check=True).stdout)


@pytest.mark.parametrize("nb,sinks,W,flags,kv_heads,G,B,lo,hi", [
    (2048, 1, 1, 0, 8, 4, 64, 16, 16),           # a long sequence, window only: as many additions as with the power term
    (2048, 1, 4, 0, 8, 4, 64, 16, 16),
    (512, 16, 4, 0, 8, 4, 64, 16, 16),
    (1024, 1, 4, POWER, 8, 4, 128, 16, 16),
    (64, 1, 1, 0, 8, 4, 64, 5, 8),               # short: between the window and 16
    (16, 1, 4, 0, 8, 4, 64, 4, 4),               # shorter: as long as an ordinary column
    (16, 1, 4, POWER, 8, 4, 64, 6, 6),           # W and the distances 4 and 8
    (1, 1, 1, 0, 1, 1, 64, 1, 16),
    (1, 0, 2 ** 31 - 1, POWER, 1, 16, 256, 1, 16),
])
def test_part_length(part, nb, sinks, W, flags, kv_heads, G, B, lo, hi):
    assert lo <= part(nb, sinks, W, flags, kv_heads, G, B) <= hi


@pytest.mark.parametrize("nb,sinks,B", [(2_000_000, 200, 64), (2_000_000, 2000, 64), (1_000_000, 500, 256), (33_554_431, 0, 64)])
def test_launch_limits(part, nb, sinks, B):
    p = part(nb, sinks, 1, 0, 1, 1, B)
    if sinks:
        assert (nb + sinks * (-(-nb // p) - 1)) * (B // 64) * 512 < 2 ** 32
    assert p >= 1
