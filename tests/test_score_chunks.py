"""The rule that cuts a prompt into the key chunks of pivot scoring (host code, no GPU): chunks are whole blocks of equal
length, never more time than chunks of 2048 keys by rounds of workgroups over the CUs, and within the workspace bound."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include <cstdio>
#include "akvq_kernels.h"
int main() {
  int B, Hq, Hkv, T, W;
  while (std::scanf("%d %d %d %d %d", &B, &Hq, &Hkv, &T, &W) == 5)
    std::printf("%d %zu\n", akvq::score_chunk(B, Hq, Hkv, T, W), akvq::score_max_triples(B, Hq, Hkv, T, W));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    path = tmp_path_factory.mktemp("chunk")
    (path / "rule.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_2501_15021_amd", "csrc"), str(path / "rule.cpp"), "-o",
                    str(path / "rule")], check=True, capture_output=True)

    def run(shapes):
        text = "\n".join(" ".join(map(str, s)) for s in shapes)
        out = subprocess.run([str(path / "rule")], input=text, check=True, capture_output=True, text=True).stdout
        return [tuple(map(int, line.split())) for line in out.split("\n") if line]
    return run


LENGTHS = sorted({64, 65, 127, 128, 129, 192, 193, 258, 640, 734, 1300, 2047, 2048, 2049, 2500, 4096, 4097, 4907, 8192, 11242,
                  16384, 20000, 32768, 65537, 131072, 200000, *range(256, 40000, 1237)})


@pytest.mark.parametrize("Hq,Hkv", [(1, 1), (32, 32), (40, 40), (14, 7), (12, 4), (32, 8), (12, 2), (28, 4), (64, 8), (8, 1)])
def test_chunks(rule, Hq, Hkv):
    shapes = [(B, Hq, Hkv, T, 64) for B in [1, 2, 3, 4, 5, 7, 8, 10, 13, 16, 20, 23, 25, 30, 32, 40, 46, 50, 63, 64, 65, 80, 100, 128]
              for T in LENGTHS]
    up = lambda a, b: -(-a // b)  # noqa: E731
    for (B, _, _, T, _), (chunk, triples) in zip(shapes, rule(shapes)):
        n, coarse, units = up(T, chunk), up(T, 2048), B * Hkv
        assert chunk % 64 == 0 and 64 <= chunk <= 2048
        assert n == coarse or (n <= 64 and chunk >= 128 and units * n <= 1024), (B, T, chunk)
        assert chunk == 2048 or chunk == up(up(T, n), 64) * 64, (B, T, chunk)  # equal lengths
        assert triples >= B * Hq * n, (B, T, chunk)
        if Hq // Hkv >= 4:  # one workgroup per CU at a time; the staging of the rows takes as long as 192 keys
            whole = min(up(T, 64) * 64, 2048)
            assert up(units * n, 256) * (min(chunk, whole) + 192) <= up(units * coarse, 256) * (whole + 192), (B, T, chunk)


def test_other_windows_keep_their_chunks(rule):
    shapes = [(1, 32, 32, 640, 16), (1, 28, 4, 4096, 32), (1, 36, 4, 4096, 64), (2, 8, 8, 100000, 48)]
    assert [c for c, _ in rule(shapes)] == [2048] * 4
