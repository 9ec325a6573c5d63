// gemm_fp8_fused.hpp -- the row/column-scaled e4m3 GEMM of few tiles as one
// kernel: scales, codes and products, with no operand planes.
//
// A block of kWaves waves computes one 32 x 32 tile of C.  The waves share
// K in steps of 64 (wave w the steps w, w + kWaves, ...); lane l = 32 h + c
// holds the step's k = 32 h .. 32 h + 31 of row c of A and of column c of B,
// as they come from memory in FP32.
//   1. Each lane takes the largest magnitudes of its row and its column; the
//      halves and waves meet in LDS, which gives every lane the scales of its
//      row and column.
//   2. The values are scaled, encoded and multiplied, 32 x 32 x 64 a step.
//      A wave's first step is still in its registers (all of K up to
//      64 kWaves); later steps are read again, from the caches.
//   3. The waves' partial tiles are added in LDS in wave order, scaled and
//      stored.
// The codes are those of the operand passes (the same magnitudes, division,
// product and encoder), so only the order of the FP32 additions over K
// differs, and that by the shape alone.
//
// The three launches of the plane form take 15-17 us whatever the size, of
// which few-tile shapes compute for 1-2 (64^3 17.4 -> 7.5 us here, 512^3
// 17.4 -> 10.0, 4429 x 19 x 18 17.4 -> 7.6).  What bounds this form is reading
// each operand once per tile of the other, a word at a time along B, and a
// second time, without loads in flight ahead, beyond 64 kWaves of K.
#pragma once
#include "common.hpp"
#include "gemm_f32.hpp"
#include "layouts.hpp"
#include "lowp.hpp"
#include "mfma.hpp"
#include "view.hpp"

namespace desc {
namespace gemm_fp8 {

constexpr int kFusedWaves = 16, kFusedTile = 32, kFusedStep = 64;
// Strides it accepts: 32-bit byte offsets over 32 rows of A or 64 rows of B.
constexpr int64_t kFusedMaxLd = int64_t(1) << 23;

struct FusedLds {
  float part[kFusedWaves][16][64];            // partial tiles
  float max_a[kFusedWaves][32], max_b[kFusedWaves][32];
  float row_max[32];                          // the tile's row maxima
};

__device__ __forceinline__ void fused_tile(const GemmProblemF32& p, idx_t tm, idx_t tn,
                                           FusedLds& lds) {
  typedef float words4 __attribute__((ext_vector_type(4))) __attribute__((aligned(4)));
  constexpr int WK = kFusedWaves, S = kFusedStep;
  auto thread = thread_x<64 * WK>();
  const int lane = (int)lane_of_wave().index(), half = lane / 32, c32 = lane % 32;
  const int w = __builtin_amdgcn_readfirstlane((int)wave_of_block<64 * WK>().index());
  const idx_t m0 = tm * kFusedTile, n0 = tn * kFusedTile;

  // The lane's byte offsets in a step: 32 consecutive k of its row of A, and
  // 32 rows of B at its column (rows and columns past the edge read the last
  // one; their results are not stored).
  auto a_g = matrix(p.A, p.M, p.lda);
  auto b_g = matrix(p.B, p.K, p.ldb);
  const BufferWindow<4> win_a{(uint32_t)p.lda, kFusedTile, S};
  const BufferWindow<4> win_b{(uint32_t)p.ldb, S, (int32_t)p.N};
  const uint32_t off_a = win_a.row((int32_t)layout::clamped_row(c32, p.M - m0)) +
                         win_a.col_valid(32 * half);
  const uint32_t off_b = win_b.row(32 * half) +
                         win_b.col_valid((int32_t)layout::clamped_group<1>(n0, c32, p.N));
  float a[32], b[32];
  auto load = [&](idx_t k0) {
    const char* pa = (const char*)&a_g.at(m0, k0) + off_a;
    const char* pb = (const char*)&b_g.at(k0, 0) + off_b;
    if (k0 + S <= p.K) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const words4 v = *(const words4*)(pa + 16 * e);
#pragma unroll
        for (int j = 0; j < 4; ++j) a[4 * e + j] = v[j];
      }
#pragma unroll
      for (int e = 0; e < 32; ++e) b[e] = *(const float*)(pb + win_b.row(e));
    } else {                      // the last, partial step: zeros past K
      const int left = (int)(p.K - k0) - 32 * half;
#pragma unroll
      for (int e = 0; e < 32; ++e) {
        a[e] = e < left ? *(const float*)(pa + 4 * e) : 0.f;
        b[e] = e < left ? *(const float*)(pb + win_b.row(e)) : 0.f;
      }
    }
  };
  const idx_t steps = (p.K + S - 1) / S;
  const idx_t mine = steps > w ? (steps - w + WK - 1) / WK : 0;

  // 1. magnitudes; the first step last, so that it stays in the registers
  float ma = 0.f, mb = 0.f;
  for (idx_t it = mine - 1; it >= 0; --it) {
    load((w + it * WK) * S);
#pragma unroll
    for (int e = 0; e < 32; ++e) {
      ma = fmaxf(ma, fabsf(a[e]));
      mb = fmaxf(mb, fabsf(b[e]));
    }
  }
  ma = fmaxf(ma, __shfl_xor(ma, 32, 64));
  mb = fmaxf(mb, __shfl_xor(mb, 32, 64));
  if (half == 0) {
    lds.max_a[w][c32] = ma;
    lds.max_b[w][c32] = mb;
  }
  sync(thread);
  ma = mb = 0.f;
#pragma unroll
  for (int x = 0; x < WK; ++x) {
    ma = fmaxf(ma, lds.max_a[x][c32]);
    mb = fmaxf(mb, lds.max_b[x][c32]);
  }
  if (w == 0 && half == 0) lds.row_max[c32] = ma;
  const float inv_a = ma > 0.f ? 448.0f / ma : 1.0f, inv_b = mb > 0.f ? 448.0f / mb : 1.0f;

  // 2. codes and products
  mfma::f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  for (idx_t it = 0; it < mine; ++it) {
    if (it > 0) load((w + it * WK) * S);
    mfma::i32x8 qa, qb;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      qa[e] = (int)lowp::e4m3x4(a[4 * e] * inv_a, a[4 * e + 1] * inv_a, a[4 * e + 2] * inv_a,
                                a[4 * e + 3] * inv_a);
      qb[e] = (int)lowp::e4m3x4(b[4 * e] * inv_b, b[4 * e + 1] * inv_b, b[4 * e + 2] * inv_b,
                                b[4 * e + 3] * inv_b);
    }
    // positions past K have code 0 (their product with the scale need not be)
    const idx_t k0 = (w + it * WK) * S;
    if (k0 + S > p.K) {
      const int left = (int)(p.K - k0) - 32 * half;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int n = left - 4 * e;              // codes of word e to keep
        const int keep = n >= 4 ? -1 : n <= 0 ? 0 : (1 << (8 * n)) - 1;
        qa[e] &= keep;
        qb[e] &= keep;
      }
    }
    acc = mfma::fp8_32x32x64(qa, qb, acc);
  }

  // 3. the sum over the waves: wave w takes accumulator register w
  static_assert(WK == 16, "one accumulator register a wave");
#pragma unroll
  for (int r = 0; r < 16; ++r) lds.part[w][r][lane] = acc[r];
  sync(thread);
  float v = lds.part[0][w][lane];
#pragma unroll
  for (int x = 1; x < WK; ++x) v += lds.part[x][w][lane];
  const int r = mfma::acc_row(w, lane);
  const idx_t row = m0 + r, col = n0 + c32;
  if (row < p.M && col < p.N)
    matrix(p.C, p.M, p.ldc).at(row, col) = (v * (lds.row_max[r] / 448.0f)) * (mb / 448.0f);
}

}  // namespace gemm_fp8
}  // namespace desc
