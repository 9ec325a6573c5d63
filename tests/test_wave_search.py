"""The 64-way search of a nondecreasing array that the segmented and grouped
kernels make with one wave, replayed on the host with their own steps against
the binary search: sizes around the powers of 64, repeated starts (empty
segments) at both ends and between, every index of the array's range."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2305_03448_amd", "csrc")

CHECK = r'''
#include <cstdio>
#include <vector>
#include "layouts.hpp"
using namespace desc;

static idx_t wave_search(const std::vector<idx_t>& start, idx_t G, idx_t t) {
  layout::Search64 s{0, G};
  int rounds = 0;
  while (!s.done()) {
    int le = 0;
    bool prefix = true;
    for (int lane = 0; lane < 64; ++lane) {
      const idx_t i = s.entry(lane);
      const bool in = i < s.hi && start[i] <= t;
      if (i < s.hi && (i < 0 || i >= G)) return -1;      // an entry outside the array
      if (in && !prefix) return -2;                      // the lanes are no prefix
      prefix = prefix && in;
      le += in;
    }
    s = s.next(le);
    if (++rounds > 4) return -3;                         // 64^4 entries
  }
  return s.lo;
}

static bool check(idx_t G, int pattern) {
  std::vector<idx_t> start(G + 1);
  idx_t at = 0;
  for (idx_t g = 0; g < G; ++g) {
    start[g] = at;
    const bool empty = pattern == 1 ? g % 3 != 1 : pattern == 2 ? g < G / 2 : pattern == 3 ? g > G / 2 : false;
    at += empty ? 0 : 1 + (g * 7) % 3;
  }
  start[G] = at;
  for (idx_t t = 0; t < at; ++t) {
    const idx_t s = wave_search(start, G, t);
    if (s != layout::seg_of_unit(start, G, t)) return false;
    if (!(start[s] <= t && t < start[s + 1])) return false;
  }
  return true;
}

int main() {
  bool ok = true;
  for (idx_t G : {1, 2, 63, 64, 65, 127, 128, 129, 4095, 4096, 4097, 16384})
    for (int p = 0; p < 4; ++p) ok = ok && check(G, p);
  std::puts(ok ? "OK" : "FAIL");
  return !ok;
}
'''


def test_wave_search_equals_the_binary_search(tmp_path):
    src, exe = str(tmp_path / "c.cpp"), str(tmp_path / "c")
    with open(src, "w") as f:
        f.write(CHECK)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, src, "-o", exe], check=True)
    assert subprocess.run([exe], capture_output=True, text=True, timeout=120).stdout == "OK\n"
