"""Transposes of matrices that are not whole tiles of aligned groups: the tile
and group starts on the host, and every element size on the GPU at the edges
of its tiles, bit for bit."""
import os
import subprocess

import pytest
import torch

import paper_2305_03448_amd as desc
from gpu_util import case, needs_gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2305_03448_amd", "csrc")

CHECK = r'''
#include <cstdio>
#include <vector>
#include "layouts.hpp"
using namespace desc;
// Every element of [0, n) is in some tile's group, and every group of a tile
// lies inside the tile and the tile inside [0, n).
template <int T, int kV>
static bool covers() {
  for (idx_t n = kV; n <= 3 * T + 5; ++n) {
    std::vector<int> seen(n, 0);
    for (idx_t t = 0; t < (n + T - 1) / T; ++t) {
      const idx_t s = layout::tile_start<T, kV>(t, n);
      const int h = (int)(n - s < T ? n - s : T);
      if (s < 0 || h < kV) return false;
      for (int x = 0; x < T / kV; ++x) {
        const int g = layout::tile_group<kV>(x, h);
        if (g < 0 || g + kV > h) return false;
        if (kV * x < h)
          for (int k = 0; k < kV; ++k) seen[s + g + k] = 1;
      }
    }
    for (int v : seen) if (!v) return false;
  }
  return true;
}
int main() {
  const bool ok = covers<128, 16>() && covers<64, 16>() && covers<128, 8>() && covers<64, 8>() &&
                  covers<32, 4>() && covers<64, 4>() && covers<128, 4>() && covers<64, 2>();
  std::puts(ok ? "OK" : "FAIL");
  return !ok;
}
'''


def test_any_shape_starts_cover_every_element(tmp_path):
    src, exe = str(tmp_path / "c.cpp"), str(tmp_path / "c")
    with open(src, "w") as f:
        f.write(CHECK)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, src, "-o", exe], check=True)
    assert subprocess.run([exe], capture_output=True, text=True, timeout=60).stdout == "OK\n"


DTYPES = {1: torch.uint8, 2: torch.int16, 4: torch.int32, 8: torch.int64}


@pytest.mark.gpu
@needs_gpu
@pytest.mark.parametrize("elem", [1, 2, 4, 8])
def test_transpose_any_shape(elem):
    v = 16 // elem
    for batch, rows, cols, off in [
            (1, v, v, 0), (1, v, 3 * v + 1, 0), (3, 63, 65, 1), (2, 127, 129, 0), (1, 128, 128, 1),
            (2, 128 + v - 1, 257, 0), (1, 128 + v - 1, 256 + v, 3), (5, 333, 250, 0),
            (1, 2500, 3700, 0), (1, 4096, 1500, 0), (1, v - 1, 200, 0), (2, 300, 1, 0)]:
        if rows == 0:
            continue
        case(f"transpose {elem}-byte {batch}x{rows}x{cols} offset {off}")
        n = batch * rows * cols
        raw = torch.randint(0, 256, ((n + off) * elem,), dtype=torch.uint8, device="cuda")
        x = raw.view(DTYPES[elem])[off:].view(batch, rows, cols)
        buf = torch.zeros(n + off + 8, dtype=DTYPES[elem], device="cuda")
        y = buf[off:off + n].view(batch, cols, rows)
        desc.desc_transpose_batched(x, y)
        assert torch.equal(y, x.transpose(1, 2))
        assert int(buf[:off].abs().sum()) == 0 and int(buf[off + n:].abs().sum()) == 0
