"""How long a workgroup of the one-pass pivot scoring waits for its head's other chunks (host code, no GPU): looks are counted
for a row of workgroups whose siblings never come, and for one whose siblings come late once."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include <cstdio>
#include "akvq_kernels.h"
// the control flow of a workgroup that goes through `heads` heads of n chunks; present(head): its siblings' words are there at once
template <typename F>
static long looks_of(int heads, int n, int own, F present, long *scored, long *first) {
  akvq::OnceWait wait;
  long looks = 0;
  *scored = 0;
  for (int h = 0; h < heads; ++h) {
    uint64_t missing = present(h) ? 0 : (n < 64 ? (1ull << n) - 1 : ~0ull) & ~(1ull << own);
    for (;;) {
      if (missing == 0) break;
      while (wait.look_again()) ++looks;
      wait.give_up();
      const int c = akvq::once_chunk_to_score(missing, own);
      if (c < 0 || c >= n || !((missing >> c) & 1)) return -1;
      if (*scored == 0) *first = c;
      missing &= ~(1ull << c);
      ++*scored;
    }
    wait.next_head();
  }
  return looks;
}
int main() {
  int heads, n, own, late;  // late: the one head whose siblings do not come (-1: none ever come)
  while (std::scanf("%d %d %d %d", &heads, &n, &own, &late) == 4) {
    long scored, first = -1;
    const long looks = looks_of(heads, n, own, [=](int h) { return late >= 0 && h != late; }, &scored, &first);
    std::printf("%ld %ld %ld %d %d\n", looks, scored, first, akvq::kOncePolls, akvq::kOnceFewPolls);
  }
}
"""


@pytest.fixture(scope="module")
def waits(tmp_path_factory):
    path = tmp_path_factory.mktemp("wait")
    (path / "wait.cpp").write_text(SOURCE)

    def run(cases, *flags):
        subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", *flags,
                        "-I" + os.path.join(ROOT, "paper_2501_15021_amd", "csrc"), str(path / "wait.cpp"), "-o", str(path / "wait")],
                       check=True, capture_output=True)
        text = "\n".join(" ".join(map(str, c)) for c in cases)
        out = subprocess.run([str(path / "wait")], input=text, check=True, capture_output=True, text=True).stdout
        return [tuple(map(int, line.split())) for line in out.split("\n") if line]
    return run


def test_a_row_without_siblings(waits):
    cases = [(heads, n, own, -1) for heads in (1, 2, 40) for n in (2, 3, 32, 33, 63, 64) for own in sorted({0, 1, n // 2, n - 1})]
    for (heads, n, own, _), (looks, scored, first, most, few) in zip(cases, waits(cases)):
        assert scored == heads * (n - 1)  # each missing chunk once
        assert looks == most + (heads - 1) * few  # one long wait, not one for every chunk or head
        assert first == (own + 1) % n  # every workgroup begins with another chunk


def test_patience_returns(waits):
    (looks, scored, _, most, few), (again, *_) = waits([(3, 5, 2, 0), (2, 5, 2, 1)])
    assert scored == 4 and looks == most and again == most
    assert few < most


def test_a_build_that_does_not_wait(waits):
    for looks, scored, _, most, few in waits([(7, 6, 3, -1)], "-DAKVQ_ONCE_POLLS=0"):
        assert looks == most == few == 0 and scored == 35
