"""The rule that lets an append's groups of four blocks run on from unit to unit (host code, no GPU): its borders, the blocks of
every unit found again by the reciprocal, and which of the shapes of test_gpu_append_flat.py it takes."""
import os
import subprocess

import pytest
import test_gpu_append_flat as flat

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include <cstdio>
#include "akvq_kernels.h"
int main() {
  long units, n_blk, window;
  while (std::scanf("%ld %ld %ld", &units, &n_blk, &window) == 3) {
    const bool on = akvq::append_runs_on(units, (int)n_blk, window != 0);
    // the unit of a block: the first and last blocks of the first, middle and last units
    const uint64_t r = akvq::reciprocal_of_blocks((int)n_blk);
    bool found = true;
    for (long unit : {0l, 1l, units / 2, units - 2, units - 1})
      for (long blk : {0l, 1l, n_blk - 1})
        if (unit >= 0 && blk < n_blk) found = found && (long)((uint64_t)(uint32_t)(unit * n_blk + blk) * r >> 32) == unit;
    std::printf("%d %d\n", on, on && !found);
  }
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    path = tmp_path_factory.mktemp("runs")
    (path / "rule.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_2501_15021_amd", "csrc"), str(path / "rule.cpp"), "-o",
                    str(path / "rule")], check=True, capture_output=True)

    def run(shapes):
        text = "\n".join(" ".join(map(str, s)) for s in shapes)
        out = subprocess.run([str(path / "rule")], input=text, check=True, capture_output=True, text=True).stdout
        lines = [tuple(map(int, line.split())) for line in out.split("\n") if line]
        assert all(lost == 0 for _, lost in lines)  # where it applies every block is found again
        return [on for on, _ in lines]
    return run


def test_borders(rule):
    # above two workgroups per CU (2 x groups x units), a twelfth of the wavefronts idle, no window, more than one block
    assert rule([(256, 2, 0), (257, 2, 0), (257, 2, 1), (600, 1, 0), (600, 4, 0), (300, 8, 0)]) == [0, 1, 0, 0, 0, 0]
    assert rule([(300, n, 0) for n in (33, 34, 37, 23, 22, 21)]) == [1, 0, 0, 0, 1, 1]
    # up to five rounds a round less (720 workgroups to 540: three both; 800 to 500; 1280 to 1120 and 1040: five both)
    assert rule([(120, 9, 0), (200, 5, 0), (160, 14, 0), (160, 13, 0)]) == [0, 1, 0, 0]
    # up to ten a round less and more than an eighth idle (six to five: 2 of 16 and 3 of 16; six both; ten to nine: 2 of 16, 3 of 16)
    assert rule([(161, 14, 0), (161, 13, 0), (152, 17, 0), (320, 14, 0), (320, 13, 0), (321, 14, 0)]) == [0, 1, 0, 0, 1, 1]
    # three blocks: three rounds to two, not four to three nor seven to six, and beyond ten rounds; seven blocks: one idle of a unit
    assert rule([(264, 3, 0), (472, 3, 0), (880, 3, 0), (1280, 3, 0), (1281, 3, 0), (340, 7, 0), (641, 7, 0)]) == [1, 0, 0, 0, 1, 0, 1]


def test_every_unit_is_found(rule):
    on = 0
    for n_blk in range(2, 40):
        most = (2 ** 32 - 1) // (n_blk * n_blk)  # units whose blocks, times n_blk, stay below 2^32
        units = [u for u in (1, 257, 300, 1000, 65535, most - 1, most, most + 1, 2 ** 31 // n_blk) if u > 0]
        got = rule([(u, n_blk, 0) for u in units])
        on += sum(got)
        assert all(not applies for u, applies in zip(units, got) if u > most)
    assert on > 80


@pytest.mark.parametrize("kind", ["plain", "rope", "tiers"])
def test_shapes_of_the_gpu_test(rule, kind):
    for cases, want in ((flat.FLAT, 1), (flat.OWN_GROUPS, 0)):
        shapes = []
        for B, H, T, _, before in cases:
            before, rows, _ = flat.rows_and_plan(B, T, before, kind)
            shapes.append((B * H, (before + rows - 1) // 32 - before // 32 + 1, 0))
        assert rule(shapes) == [want] * len(cases), (kind, shapes)
