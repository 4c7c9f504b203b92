"""The rule that chooses how a prompt's pivots are scored (host code, no GPU): what each kernel takes, and that a workspace of
akvq_select_workspace_bytes holds what the chosen one keeps there, for the shape itself and for every smaller one."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include <cstdio>
#include "akvq_kernels.h"
int main() {
  int B, Hq, Hkv, T, W, shared;
  float scale;
  while (std::scanf("%d %d %d %d %d %f %d", &B, &Hq, &Hkv, &T, &W, &scale, &shared) == 7)
    std::printf("%d %zu %zu %zu\n", akvq::score_path(B, Hq, Hkv, T, W, scale, shared), akvq::score_head_masses(B, Hq, Hkv, T),
                akvq::score_max_triples(B, Hq, Hkv, T, W), akvq::score_max_head_masses(B, Hq, Hkv, T, W));
}
"""
TWO, SMALL, ONCE = 0, 1, 2


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    path = tmp_path_factory.mktemp("path")
    (path / "rule.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_2501_15021_amd", "csrc"), str(path / "rule.cpp"), "-o",
                    str(path / "rule")], check=True, capture_output=True)

    def run(shapes):
        text = "\n".join(" ".join(map(str, s)) for s in shapes)
        out = subprocess.run([str(path / "rule")], input=text, check=True, capture_output=True, text=True).stdout
        return [tuple(map(int, line.split())) for line in out.split("\n") if line]
    return run


LENGTHS = sorted({64, 65, 127, 255, 256, 257, 300, 511, 512, 513, 767, 768, 769, 1023, 1024, 1025, 2048, 3001, 8192, 16384, 16385, 32767, 32768,
                  32769, 40000, 131072})
BATCHES = [1, 2, 3, 4, 5, 7, 8, 9, 13, 16, 17, 19, 32, 33, 64, 65, 73, 128, 129, 146, 300]


@pytest.mark.parametrize("Hq,Hkv", [(1, 1), (32, 32), (40, 40), (16, 8), (32, 8), (12, 2), (28, 4), (64, 8), (8, 1), (9, 1)])
def test_paths(rule, Hq, Hkv):
    shapes = [(B, Hq, Hkv, T, 64, 0.1, shared) for shared in (0, 1) for T in LENGTHS for B in BATCHES]
    most = {}
    for (B, _, _, T, _, _, shared), (path, masses, triples, max_masses) in zip(shapes, rule(shapes)):
        chunks, heads = -(-T // 512), B * Hq
        if path == SMALL:
            assert T <= 768 and not shared
        if path == ONCE:
            assert chunks <= 64 and triples >= heads * chunks
            assert Hq == Hkv or (heads * chunks <= 512 and not shared)  # several heads: all workgroups resident at once
        assert Hq <= 8 * Hkv or path == TWO
        if path != TWO and Hq > Hkv:
            assert masses == heads * (-(-T // 4) * 4) and max_masses >= masses
        if not shared:
            most[B, T] = (triples, max_masses)
    for (B, T), sizes in most.items():  # a workspace of the largest batch and prompt serves all smaller ones
        assert all(x <= y for x, y in zip(sizes, most[BATCHES[-1], T])) and all(x <= y for x, y in zip(sizes, most[B, LENGTHS[-1]]))


def test_what_takes_two_passes(rule):
    cases = [(1, 32, 32, 300, 48, 0.1, 0), (1, 32, 32, 300, 64, 0.0, 0), (1, 32, 32, 300, 64, -0.1, 0), (1, 32, 32, 300, 64, 0.1, 1),
             (1, 28, 4, 300, 64, 0.1, 1), (1, 32, 32, 32769, 64, 0.1, 0), (64, 32, 8, 768, 64, 0.1, 0)]
    assert [r[0] for r in rule(cases)] == [TWO] * len(cases)
    # one head per KV head: up to 64 workgroups and four chunks
    few = [(1, 32, 32, 1024, 64, 0.1, 0), (33, 1, 1, 1024, 64, 0.1, 0), (1, 2, 2, 2048, 64, 0.1, 0), (1, 2, 2, 2049, 64, 0.1, 0), (1, 16, 16, 2048, 64, 0.1, 1),
           (17, 1, 1, 2048, 64, 0.1, 1)]
    assert [r[0] for r in rule(few)] == [TWO, ONCE, TWO, ONCE, TWO, ONCE]
    assert [r[0] for r in rule([(1, 32, 32, 640, 64, 0.1, 0), (17, 32, 32, 640, 64, 0.1, 0), (8, 32, 32, 16384, 64, 0.1, 1)])] == [SMALL, ONCE, ONCE]
