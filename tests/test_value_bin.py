"""The histograms' bin of a value, compiled for the CPU from the kernels' source with the conversions to an integer
checked: every value has a bin (or none, below or above the range), a value that is no number the first one."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
int main() {
  const double inf = INFINITY, big = 1.7e308;
  const double values[] = {NAN, -NAN, -inf, inf, -big, big, 0.0, -0.0, 1e-320, 0.1, 0.25, 0.5, 0.9999999999999999, 1.0, -0.1};
  const double ranges[][2] = {{0.0, 1.0}, {-0.1, 0.3}, {-big, big}, {-1e-320, 1e-320}, {0.25, 0.25000000000000006}};
  for (const auto& r : ranges)
    for (int nb : {1, 2, 200, 1024, 65536})
      for (double v : values) {
        const int b = value_bin(v, r[0], r[1], nb);
        const bool ok = v < r[0] ? b == -1 : (v >= r[1] ? b == nb : (v != v ? b == 0 : b >= 0 && b < nb));
        if (!ok) {
          std::printf("%g in [%g, %g) of %d: %d\n", v, r[0], r[1], nb, b);
          return 1;
        }
      }
  return 0;
}
"""


def test_every_value_has_a_defined_bin(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    with open(os.path.join(ROOT, "paper_1110_4894_amd", "csrc", "rt_kernels.hip")) as f:
        body = re.search(r"__device__ __forceinline__ (int value_bin\(.*?\n\})", f.read(), re.S).group(1)
    src, exe = tmp_path / "bin.cpp", tmp_path / "bin"
    src.write_text("#include <cmath>\n#include <cstdio>\n#include <initializer_list>\nusing std::floor;\nstatic " + body + MAIN)
    subprocess.run([gxx, "-std=c++17", "-O1", "-fsanitize=undefined,float-cast-overflow", "-fno-sanitize-recover=all",
                    str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
