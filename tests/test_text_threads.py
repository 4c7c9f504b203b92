"""How many threads list the text positions of a row (host code, no GPU): the borders of the rule."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include <cstdio>
#include "akvq_kernels.h"
int main() {
  long rows;
  int T;
  while (std::scanf("%ld %d", &rows, &T) == 2) std::printf("%d\n", akvq::text_threads(rows, T));
}
"""


def test_borders(tmp_path):
    (tmp_path / "rule.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_2501_15021_amd", "csrc"), str(tmp_path / "rule.cpp"), "-o", str(tmp_path / "rule")],
                   check=True, capture_output=True)
    cases = [(1, 1), (1, 4097), (28, 8192), (28, 8193), (256, 8193), (257, 8193), (288, 4708), (352, 20425), (2048, 8192), (1, 2147483647), (65535, 2147483647)]
    out = subprocess.run([str(tmp_path / "rule")], input="\n".join(f"{r} {t}" for r, t in cases), check=True, capture_output=True, text=True).stdout
    assert [int(x) for x in out.split()] == [256, 256, 256, 1024, 1024, 256, 256, 256, 256, 1024, 256]
