// gemm_direct.hpp -- FP32 matrix-core tiles whose operands go straight from
// memory to the matrix instructions, without LDS staging and without
// barriers in the K loop.
//
// A wave holds a (16 FM) x (16 FN) part of C as FM x FN fragments of 16 x 16
// and takes K in stages, of 16 for FP32 products.  Lane l = 16 q + c (q = 0..3, c = 0..15)
// carries the stage's k = 4 q + kk at step kk, for A and for B alike, so
//   A : four consecutive k of row m0 + 16 i + c are one 16-byte load, and
//   B : FN consecutive columns of row k, from n0 + FN c, are one load of
//       FN words; fragment j of lane c is column n0 + FN c + j.
// Four lanes read 64 consecutive bytes of a row of A and sixteen lanes the
// whole width of the tile from a row of B, and a lane's results are FN
// consecutive columns of C, stored together.
//
// kWK waves share one tile and take its stages in turn (wave w the stages w,
// w + kWK, ...); their partial sums meet in LDS and are added in wave order,
// so the result depends on the shape only.  Without a staging buffer a tile
// can be as small as the shape asks for: 1000 x 1500 x 777 takes 25 us as 256
// tiles of 64 x 96 against 92 us as 96 LDS-staged tiles of 128 x 128 (whose
// rows, 777 words, it loads one by one), 32 x 4096 x 4096 18.7 us against 154,
// 64 x 64 x 4096 11.9 against 123, 512^3 6.4 against 19.5.
//
// Edges without branches: a row past M reads row M - 1 (its results are not
// stored); a column group that would cross N starts at N - FN instead, for
// the loads and the stores alike, so every group is whole and two groups may
// compute and store the same value twice.  Only the last, partial stage of K
// masks its elements, in A and in B (so that no 0 * Inf enters a sum).
// Loads need 4-byte alignment only.
#pragma once
#include "common.hpp"
#include "gemm_f32.hpp"
#include "layouts.hpp"
#include "lowp.hpp"
#include "mfma.hpp"
#include "view.hpp"

namespace desc {

// kFM x kFN fragments a wave, kWM x kWN wave tiles a block, kWK waves to each
// tile's K, kDepth stages of loads in flight per wave.
template <int kFM, int kFN, int kWM, int kWN, int kWK, int kDepth>
struct DirectCfg {
  static constexpr int fm = kFM, fn = kFN, wm = kWM, wn = kWN, wk = kWK, depth = kDepth;
  static constexpr int threads = 64 * kWM * kWN * kWK;
  static constexpr int wtm = 16 * kFM, wtn = 16 * kFN;       // wave tile
  static constexpr int bm = wtm * kWM, bn = wtn * kWN;       // block tile
  // the waves' partial tiles, when more than one shares a tile
  static constexpr int lds_floats = kWK > 1 ? kWM * kWN * kWK * wtm * wtn : 4;
  static_assert(kFN >= 1 && kFN <= 4, "one load holds a lane's columns");
};

// Strides the direct form accepts: its 32-bit byte offsets span at most 64
// rows of A, or 32 rows of B (16 in FP32 products) and one row's columns.
constexpr int64_t kDirectMaxLd = int64_t(1) << 23;

namespace gemm_direct {

// kN consecutive floats at 4-byte alignment.
template <int kN>
struct Words {
  typedef float t __attribute__((ext_vector_type(kN))) __attribute__((aligned(4)));
};
template <>
struct Words<1> {
  typedef float t;
};

// One tile of C = A * B at block tile (tm, tn).  `lds` holds
// C::lds_floats floats (unused when one wave takes all of K).
//
// kSplit: the three-product split-BF16 arithmetic.  A stage is then 32 values
// of K, eight consecutive ones a lane (k = 8 q + kk, two 16-byte loads of a
// row of A, eight rows of B), split into hi and lo in registers as they are
// used, for 16 x 16 x 32 bfloat16 instructions on the same lanes.
template <class C, bool kSplit = false>
__device__ __forceinline__ void tile(const GemmProblemF32& p, idx_t tm, idx_t tn, float* lds) {
  constexpr int FM = C::fm, FN = C::fn, WK = C::wk, D = C::depth;
  constexpr int BK = kSplit ? 32 : 16, QK = BK / 4;      // k per stage and per lane
  using awords = typename Words<4>::t;
  using bwords = typename Words<FN>::t;
  auto thread = thread_x<C::threads>();
  const int lane = (int)lane_of_wave().index();
  const int quarter = lane / 16, c16 = lane % 16;
  const int w = __builtin_amdgcn_readfirstlane((int)wave_of_block<C::threads>().index());
  const int wk = w % WK, part = w / WK;                  // K share, wave tile of the block
  const idx_t m0 = tm * C::bm + part / C::wn * C::wtm;
  const idx_t n0 = tn * C::bn + part % C::wn * C::wtn;

  // The lane's byte offsets in a stage, from the wave tile's first row of A
  // (the last row of A when the whole wave tile lies past it) and from row
  // k0 of B.
  auto a_g = matrix(p.A, p.M, p.lda);
  auto b_g = matrix(p.B, p.K, p.ldb);
  const BufferWindow<4> win_a{(uint32_t)p.lda, C::wtm, BK};
  const BufferWindow<4> win_b{(uint32_t)p.ldb, BK, (int32_t)p.N};
  const idx_t a_row0 = m0 < p.M ? m0 : p.M - 1;
  const auto a_first = array(&a_g.at(a_row0, 0), p.K);
  const idx_t col = layout::clamped_group<FN>(n0, c16, p.N);
  uint32_t off_a[FM], off_b[QK];
#pragma unroll
  for (int i = 0; i < FM; ++i)
    off_a[i] = win_a.row((int32_t)layout::clamped_row(16 * i + c16, p.M - a_row0)) +
               win_a.col_valid(layout::gemm16_frag_k<BK>(quarter));
#pragma unroll
  for (int kk = 0; kk < QK; ++kk)
    off_b[kk] = win_b.row(layout::gemm16_frag_k<BK>(quarter) + kk) + win_b.col_valid((int32_t)col);

  struct Stage {
    f32x4 a[FM][QK / 4];
    float b[QK][FN];
  };
  // this wave's whole stages: wk, wk + WK, ... below K / BK
  const idx_t whole = p.K / BK;
  const idx_t mine = whole > wk ? (whole - wk + WK - 1) / WK : 0;
  auto load = [&](idx_t it, Stage& s) {
    const idx_t k0 = (wk + it * WK) * BK;
    const char* pa = (const char*)&a_first[k0];
    const char* pb = (const char*)&b_g.at(k0, 0);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int h = 0; h < QK / 4; ++h) s.a[i][h] = *(const awords*)(pa + off_a[i] + 16 * h);
#pragma unroll
    for (int kk = 0; kk < QK; ++kk) {
      const bwords v = *(const bwords*)(pb + off_b[kk]);
      if constexpr (FN == 1) {
        s.b[kk][0] = v;
      } else {
#pragma unroll
        for (int j = 0; j < FN; ++j) s.b[kk][j] = v[j];
      }
    }
  };
  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](const Stage& s) {
    if constexpr (kSplit) {
      // hi and lo of eight values of k, packed for one operand register group
      auto split8 = [](auto&& value, u32x4& hi, u32x4& lo) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const lowp::Split2 p2 = lowp::split_bf16x2(value(2 * e), value(2 * e + 1));
          hi[e] = p2.hi;
          lo[e] = p2.lo;
        }
      };
      u32x4 bh[FN], bl[FN];
#pragma unroll
      for (int j = 0; j < FN; ++j) split8([&](int k) { return s.b[k][j]; }, bh[j], bl[j]);
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        u32x4 ah, al;
        split8([&](int k) { return s.a[i][k / 4][k % 4]; }, ah, al);
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          acc[i][j] = mfma::bf16_16x16x32(al, bh[j], acc[i][j]);
          acc[i][j] = mfma::bf16_16x16x32(ah, bl[j], acc[i][j]);
          acc[i][j] = mfma::bf16_16x16x32(ah, bh[j], acc[i][j]);
        }
      }
    } else {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j)
            acc[i][j] = mfma::f32_16x16x4(s.a[i][0][kk], s.b[kk][j], acc[i][j]);
    }
  };

  // D stages in flight: stage it + D is loaded into the registers of stage
  // it as soon as its matrix ops are issued.
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
  // fewer than 2 D stages left, the first D of them loaded
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (it + d < mine) {
      compute(st[d]);
      if (it + d + D < mine) load(it + d + D, st[d]);
    }
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (it + D + d < mine) compute(st[d]);
  // the last, partial stage, by the wave whose turn it is
  if (p.K % BK != 0 && wk == (int)(whole % WK)) {
    Stage s;
    const idx_t k0 = whole * BK;
    const int left = (int)(p.K - k0), k = layout::gemm16_frag_k<BK>(quarter);
    const char* pa = (const char*)&a_first[k0];
    const char* pb = (const char*)&b_g.at(k0, 0);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int e = 0; e < QK; ++e)
        s.a[i][e / 4][e % 4] = k + e < left ? *(const float*)(pa + off_a[i] + 4 * e) : 0.f;
#pragma unroll
    for (int kk = 0; kk < QK; ++kk)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        s.b[kk][j] = k + kk < left ? *(const float*)(pb + off_b[kk] + 4 * j) : 0.f;
    compute(s);
  }

  // Register r of fragment (i, j) is row 16 i + 4 quarter + r, column j of
  // the lane's group.
  auto c_g = matrix(p.C, p.M, p.ldc);
  const bool col_in = n0 + FN * c16 < p.N;
  auto store = [&](int slot, const float (&v)[FN]) {      // slot = 4 i + r
    const idx_t row = m0 + 16 * (slot / 4) + 4 * quarter + slot % 4;
    if (row < p.M && col_in) {
      bwords o;
      if constexpr (FN == 1) {
        o = v[0];
      } else {
#pragma unroll
        for (int j = 0; j < FN; ++j) o[j] = v[j];
      }
      *(bwords*)&c_g.at(row, col) = o;
    }
  };
  if constexpr (WK == 1) {
#pragma unroll
    for (int s = 0; s < 4 * FM; ++s) {
      float v[FN];
#pragma unroll
      for (int j = 0; j < FN; ++j) v[j] = acc[s / 4][j][s % 4];
      store(s, v);
    }
  } else {
    // partial tiles as [part][wave][slot][fragment column][lane] words: each
    // access of a wave is 64 consecutive words
    auto parts = array(lds, C::lds_floats).template group<64>().template group<FN>()
                     .template group<4 * FM>().template group<WK>().idx(part);
    auto my = parts.idx(wk);
#pragma unroll
    for (int s = 0; s < 4 * FM; ++s)
#pragma unroll
      for (int j = 0; j < FN; ++j) my.at(s, j, lane) = acc[s / 4][j][s % 4];
    sync(thread);
    // wave wk adds the slots wk, wk + WK, ... of its tile
    for (int s = wk; s < 4 * FM; s += WK) {
      float v[FN];
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        v[j] = parts.at(0, s, j, lane);
#pragma unroll
        for (int x = 1; x < WK; ++x) v[j] += parts.at(x, s, j, lane);
      }
      store(s, v);
    }
  }
}

}  // namespace gemm_direct
}  // namespace desc
