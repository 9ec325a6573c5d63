// Host enumeration of the direct GEMM tile's maps (gemm_direct.hpp): every
// line "OK name" or "FAIL name".
#include <cstdio>
#include <set>
#include <utility>
#include <vector>

#include "layouts.hpp"

using namespace desc;

static int failures = 0;
static void report(const char* name, bool ok) {
  std::printf("%s %s\n", ok ? "OK" : "FAIL", name);
  failures += !ok;
}

// The blocks of a grid take every tile exactly once, and each XCD's blocks
// (block % 8, in order) a contiguous run of the tile sequence.
static bool tile_order() {
  for (idx_t tm : {1, 2, 3, 7, 8, 9, 16, 17, 63})
    for (idx_t tn : {1, 2, 5, 8, 13, 64}) {
      std::set<std::pair<idx_t, idx_t>> seen;
      for (idx_t b = 0; b < tm * tn; ++b) {
        const auto t = layout::xcd_run_tile(b, tm, tn);
        if (t.m < 0 || t.m >= tm || t.n < 0 || t.n >= tn) return false;
        if (!seen.insert({t.m, t.n}).second) return false;
      }
    }
  return true;
}

// A tile's column groups lie inside the row and together hold every column
// of the tile that exists.
template <int kN>
static bool groups() {
  for (idx_t N = kN; N <= 200; ++N)
    for (idx_t n0 = 0; n0 < N; n0 += 16 * kN) {
      std::set<idx_t> cols;
      for (int c = 0; c < 16; ++c) {
        const idx_t first = layout::clamped_group<kN>(n0, c, N);
        if (first < 0 || first + kN > N) return false;
        if (n0 + kN * c < N)                       // the lanes that store
          for (int j = 0; j < kN; ++j) cols.insert(first + j);
      }
      for (idx_t n = n0; n < N && n < n0 + 16 * kN; ++n)
        if (!cols.count(n)) return false;
    }
  return true;
}

static bool rows() {
  for (idx_t valid = 1; valid <= 64; ++valid)
    for (idx_t r = 0; r < 64; ++r) {
      const idx_t x = layout::clamped_row(r, valid);
      if (x < 0 || x >= valid || (r < valid && x != r)) return false;
    }
  return true;
}

// The stages of kWK waves, the lanes' quarters and steps, and the partial
// stage with its mask hold every k below K once.
template <int BK>
static bool k_split() {
  for (int wk : {1, 2, 4, 8, 16})
    for (idx_t K = 0; K <= 600; ++K) {
      std::vector<int> times(K, 0);
      const idx_t whole = K / BK;
      for (int w = 0; w < wk; ++w) {
        const idx_t mine = whole > w ? (whole - w + wk - 1) / wk : 0;
        for (idx_t it = 0; it < mine; ++it)
          for (int q = 0; q < 4; ++q)
            for (int kk = 0; kk < BK / 4; ++kk) {
              const idx_t k = (w + it * wk) * BK + layout::gemm16_frag_k<BK>(q) + kk;
              if (k >= K) return false;
              ++times[k];
            }
        if (K % BK != 0 && w == (int)(whole % wk))
          for (int q = 0; q < 4; ++q)
            for (int kk = 0; kk < BK / 4; ++kk) {
              const idx_t k = whole * BK + layout::gemm16_frag_k<BK>(q) + kk;
              if (k < K) ++times[k];
            }
      }
      for (int t : times)
        if (t != 1) return false;
    }
  return true;
}

int main() {
  report("tile_order", tile_order());
  report("groups_1", groups<1>());
  report("groups_2", groups<2>());
  report("groups_3", groups<3>());
  report("groups_4", groups<4>());
  report("rows", rows());
  report("k_split", k_split<16>() && k_split<32>());
  return failures != 0;
}
