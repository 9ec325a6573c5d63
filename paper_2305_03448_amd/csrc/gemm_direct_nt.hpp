// gemm_direct_nt.hpp -- the direct tile (gemm_direct.hpp) over the padded e4m3
// planes of the FP8 GEMM: fragments go straight from memory to the matrix
// instructions, and the waves of a block share a tile's K.
//
// Both planes are K-contiguous and padded with zeros to whole tiles, so there
// are no edges before the stores.  A wave holds (32 FM) x (32 FN) of C and
// takes K in stages of 128 bytes, one line of every row, as two 32 x 32 x 64
// steps: lane 32 h + c holds bytes 64 s + 32 h .. + 31 of row c of a fragment
// in step s.  Wave w of kWK takes the stages w, w + kWK, ...; the partial
// tiles meet in LDS and are added in wave order, scaled and stored.
//
// It serves shapes with few 128 x 128 tiles, whose K loop is one long chain
// in the LDS-staged form: 64 x 64 x 4096 spends 22 us there on one CU.
#pragma once
#include "common.hpp"
#include "gemm_nt.hpp"
#include "mfma.hpp"
#include "view.hpp"

namespace desc {

template <int kFM, int kFN, int kWK, int kDepth>
struct DirectNtCfg {
  static constexpr int fm = kFM, fn = kFN, wk = kWK, depth = kDepth, threads = 64 * kWK;
  static constexpr int bm = 32 * kFM, bn = 32 * kFN, bkb = 128;
  static constexpr int slots = 16 * kFM * kFN;            // accumulator registers a lane
  static constexpr int lds_floats = kWK * slots * 64;
  static_assert(slots % kWK == 0, "slots divide among the waves");
};

namespace gemm_nt {

// Rows of a tile span below 2^31 bytes (32-bit offsets).
template <class C>
__host__ __device__ inline bool direct_tile_ok(int64_t row_bytes) {
  return (C::bm > C::bn ? C::bm : C::bn) * row_bytes < (int64_t(1) << 31);
}

template <class C>
__device__ __forceinline__ void direct_tile(const NtOperands& p, idx_t tm, idx_t tn, float* lds) {
  constexpr int FM = C::fm, FN = C::fn, WK = C::wk, D = C::depth;
  auto thread = thread_x<C::threads>();
  const int lane = (int)lane_of_wave().index(), half = lane / 32, c32 = lane % 32;
  const int w = __builtin_amdgcn_readfirstlane((int)wave_of_block<C::threads>().index());
  const idx_t m0 = tm * C::bm, n0 = tn * C::bn;
  const BufferWindow<1> win{(uint32_t)p.row_bytes, C::bm > C::bn ? C::bm : C::bn,
                            (int32_t)p.row_bytes};
  const auto a_first = array(&matrix(p.a[0], 0, p.row_bytes).at(m0, 0), p.row_bytes);
  const auto b_first = array(&matrix(p.b[0], 0, p.row_bytes).at(n0, 0), p.row_bytes);
  uint32_t off_a[FM], off_b[FN];
#pragma unroll
  for (int i = 0; i < FM; ++i) off_a[i] = win.row(32 * i + c32) + win.col_valid(32 * half);
#pragma unroll
  for (int j = 0; j < FN; ++j) off_b[j] = win.row(32 * j + c32) + win.col_valid(32 * half);

  struct Stage {
    Frag<32> a[FM][2], b[FN][2];
  };
  const idx_t stages = p.row_bytes / C::bkb;
  const idx_t mine = stages > w ? (stages - w + WK - 1) / WK : 0;
  auto load = [&](idx_t it, Stage& s) {
    const idx_t k0 = (w + it * WK) * C::bkb;
    auto frag = [](const uint8_t* q, Frag<32>& f) {
      f.v0 = *(const u32x4*)q;
      f.v1 = *(const u32x4*)(q + 16);
    };
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int st = 0; st < 2; ++st) frag(&a_first[k0] + off_a[i] + 64 * st, s.a[i][st]);
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int st = 0; st < 2; ++st) frag(&b_first[k0] + off_b[j] + 64 * st, s.b[j][st]);
  };
  mfma::f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  auto compute = [&](const Stage& s) {
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = mfma::fp8_32x32x64(s.a[i][st].i8(), s.b[j][st].i8(), acc[i][j]);
  };
  Stage st[D];
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (d < mine) load(d, st[d]);
  idx_t it = 0;
  for (; it + 2 * D <= mine; it += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      compute(st[d]);
      __builtin_amdgcn_sched_barrier(0);
      load(it + d + D, st[d]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (it + d < mine) {
      compute(st[d]);
      if (it + d + D < mine) load(it + d + D, st[d]);
    }
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (it + D + d < mine) compute(st[d]);

  // partial tiles as [wave][slot][lane] words, slot = 16 (FN i + j) + r
  auto parts = matrices(lds, WK, C::slots, 64);
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) parts.at(w, 16 * (FN * i + j) + r, lane) = acc[i][j][r];
  sync(thread);
  auto c_g = matrix(p.C, p.M, p.ldc);
  auto sa = array(p.sa, 0);
  auto sb = array(p.sb, 0);
#pragma unroll 4
  for (int s = w; s < C::slots; s += WK) {
    float v = parts.at(0, s, lane);
#pragma unroll
    for (int x = 1; x < WK; ++x) v += parts.at(x, s, lane);
    const idx_t row = m0 + 32 * (s / 16 / FN) + mfma::acc_row(s % 16, lane);
    const idx_t col = n0 + 32 * (s / 16 % FN) + c32;
    if (row < p.M && col < p.N) c_g.at(row, col) = (v * sa[row]) * sb[col];
  }
}

}  // namespace gemm_nt
}  // namespace desc
