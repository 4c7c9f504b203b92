"""How the one-head decode kernel deals the units of 16-bit rows to splits and wavefronts (host code, no GPU): every unit
of the salient list and of the recent window is read once, and in a fused step the salient units and the new row's unit by
the split that appends."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include <cstdio>
#include <vector>
#include "akvq_kernels.h"
using namespace akvq;
template <int NW> int check(int n_split, int win, int T_len, int cnt, int fused) {
  DecodeArgs a{};
  a.n_split = n_split; a.win_len = win; a.T_len = T_len; a.fused_append = fused;
  for (int owner = 0; owner < (fused ? n_split : 1); ++owner) {
    std::vector<int> sal((cnt + 31) / 32), w(win / 32);
    const int fresh = ((T_len - 1) % win) / 32;
    for (int s = 0; s < n_split; ++s)
      for (int v = 0; v < NW; ++v) {
        const bool appends = fused && s == owner;
        const RowUnits u = salient_units<NW>(a, cnt, s, v, appends);
        for (int i = u.first; i < u.limit; i += u.step) {
          if (u.unit(i) < 0 || u.unit(i) >= (int)sal.size() || (fused && !appends)) return 1;
          ++sal[u.unit(i)];
        }
        const RowUnits x = window_units<NW>(a, cnt, s, v, appends);
        for (int i = x.first; i < x.limit; i += x.step) {
          if (x.unit(i) < 0 || x.unit(i) >= (int)w.size() || (fused && x.unit(i) == fresh && !appends)) return 2;
          ++w[x.unit(i)];
        }
      }
    for (int n : sal) if (n != 1) return 3;
    for (int n : w) if (n != 1) return 4;
  }
  return 0;
}
template <int NW> int check_pairs(int win, int cnt) {
  for (const int rows : {cnt, win}) {
    std::vector<int> seen((rows + 63) / 64);
    for (int v = 0; v < NW; ++v) {
      const RowUnits u = rows == cnt ? paired_units<NW>(cnt, 0, v) : paired_units<NW>(win, cnt, v);
      for (int i = u.first; i < u.limit; i += u.step) ++seen.at(i);
    }
    for (int n : seen) if (n != 1) return 5;
  }
  return 0;
}
int main() {
  for (int win : {1, 31, 64, 100, 128, 192, 512, 1024}) for (int cnt : {0, 1, 31, 32, 33, 64, 65, 200, 1121})
    if (check_pairs<4>(win, cnt)) { std::printf("pairs: window %d salient %d\n", win, cnt); return 1; }
  for (int n_split : {1, 2, 3, 5, 8, 32, 64}) for (int win : {64, 128, 192, 1024}) for (int cnt : {0, 1, 31, 32, 33, 64, 200, 1121})
    for (int T_len : {1, 2, 33, 64, 65, 100, 127, 128, 129, 3002, 20012}) for (int fused : {0, 1}) {
      const int a = check<4>(n_split, win, T_len, cnt, fused), b = check<8>(n_split, win, T_len, cnt, fused);
      if (a || b) { std::printf("%d %d: splits %d window %d salient %d rows %d fused %d\n", a, b, n_split, win, cnt, T_len, fused); return 1; }
    }
  std::puts("ok");
}
"""


def test_every_unit_once(tmp_path):
    (tmp_path / "units.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_2501_15021_amd", "csrc"), str(tmp_path / "units.cpp"), "-o",
                    str(tmp_path / "units")], check=True, capture_output=True)
    done = subprocess.run([str(tmp_path / "units")], capture_output=True, text=True)
    assert done.returncode == 0 and done.stdout.strip() == "ok", done.stdout
