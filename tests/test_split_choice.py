"""How many KV splits a decode call without a split count gets (host code, no GPU): never more than the public maximum, which
the workspace is sized for, and no more than before where the merge would cost what the splits gain."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include <cstdio>
#include "akvq_kernels.h"
using namespace akvq;
static int at(int B, int Hq, int Hkv, int T, int win, int cap, bool fused) {
  DecodeArgs a{};
  a.B = B; a.Hq = Hq; a.Hkv = Hkv; a.T_len = T; a.S_cap = cap; a.win_len = win;
  a.t_win = (((T > win ? T - win : 0) + 1) & ~1);
  if (win == 0) a.t_win = T;
  return decode_splits(a, fused);
}
#define CHECK(c) do { if (!(c)) { std::printf("%s\n", #c); return 1; } } while (0)
int main() {
  const int lengths[] = {1, 640, 1023, 1024, 1077, 1239, 1472, 1473, 1985, 2100, 3000, 5000, 20011, 40000, 131072};
  for (int B : {1, 3, 8, 16, 17, 64, 200}) for (int Hkv : {1, 2, 4, 8, 32, 40}) for (int R : {1, 2, 7, 8})
    for (int win : {0, 64, 512}) for (int cap : {64, 128, 1152}) for (bool fused : {false, true}) {
      int last = 1;
      for (int T : lengths) {
        const int n = at(B, R * Hkv, Hkv, T, win, cap, fused), most = decode_most_splits((long)B * Hkv, T);
        if (n < 1 || n > most || n < last || (B * Hkv > 64 && n != most) || (T >= 20011 && n != most) || (T < 1024 && n != 1)) {
          std::printf("B %d Hkv %d R %d T %d window %d slots %d fused %d: %d of %d after %d\n", B, Hkv, R, T, win, cap, fused, n, most, last);
          return 1;
        }
        last = n;
      }
    }
  // 28/4 heads, a step with a long window: 14.3 us in one split, 15.1 in 8; without the window 11.7 and 10.9
  CHECK(at(1, 28, 4, 1077, 512, 64, true) == 1 && at(8, 28, 4, 1500, 512, 64, true) == 1 && at(1, 28, 4, 1077, 0, 64, true) == 8);
  // ... its decode call, whose 16-bit rows all splits share
  CHECK(at(1, 28, 4, 1077, 512, 64, false) == 8 && at(1, 28, 4, 1077, 0, 64, false) == 1 && at(1, 28, 4, 1281, 0, 64, false) == 10);
  // many salient rows in a step, many units
  CHECK(at(30, 8, 1, 1100, 0, 256, true) == 1 && at(60, 8, 1, 1500, 0, 64, false) == 1 && at(16, 28, 4, 2000, 0, 64, false) == 4);
  // one head per KV head: a step's window is shared
  CHECK(at(1, 32, 32, 1024, 512, 64, true) == 8 && at(2, 32, 32, 1500, 0, 64, false) == 1 && at(2, 32, 32, 2000, 0, 64, false) == 4);
  std::puts("ok");
}
"""


def test_splits_of_a_call_without_a_count(tmp_path):
    (tmp_path / "splits.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_2501_15021_amd", "csrc"), str(tmp_path / "splits.cpp"), "-o",
                    str(tmp_path / "splits")], check=True, capture_output=True)
    done = subprocess.run([str(tmp_path / "splits")], capture_output=True, text=True)
    assert done.returncode == 0 and done.stdout.strip() == "ok", done.stdout
