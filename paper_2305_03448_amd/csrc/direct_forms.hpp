// direct_forms.hpp -- the compiled direct tiles (gemm_direct.hpp), their
// launches and the choice among them, for the plain GEMM's FP32 and
// split-BF16 modes.
//
// What bounds these kernels is the operand traffic through the CU's 32 KB
// cache: with two blocks on a CU their lines evict each other before the
// neighbouring lanes and waves have used them (FP32, 4096^3 in 128 x 128
// tiles: 1555 us with two blocks a CU, 1045 us with one; 1024 tiles of
// 64 x 64 at K = 1024: 100 against 84 us).  A long K therefore launches with
// enough LDS reserved that one block has the CU; with little to read per
// block the second block's overlap of prologue and stores wins instead
// (K = 64: 13.2 against 17.2 us), and tiles up to 32 x 32 read too little to
// disturb each other at any K measured.
#pragma once
#include <cmath>

#include "gemm_direct.hpp"
#include "launch.hpp"

namespace desc {
namespace {

constexpr size_t kOneBlockLds = 84 * 1024;          // over half of a CU's 160 KB
constexpr int64_t kOneBlockWords = 51200;           // operand words per block from which it pays

template <class C, bool kSplit>
__global__ __launch_bounds__(C::threads) void gemm_direct_kernel(
    const float* __restrict__ A, int64_t lda, const float* __restrict__ B, int64_t ldb,
    float* __restrict__ Cm, int64_t ldc, int64_t M, int64_t N, int64_t K) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const GemmProblemF32 p{A, lda, B, ldb, Cm, ldc, M, N, K};
  const auto t = layout::xcd_run_tile(block_x().index(), (M + C::bm - 1) / C::bm,
                                      (N + C::bn - 1) / C::bn);
  gemm_direct::tile<C, kSplit>(p, t.m, t.n, lds);
}

template <class C, bool kSplit>
hipError_t launch_direct(const GemmProblemF32& g, hipStream_t s) {
  const int64_t tiles = ((g.M + C::bm - 1) / C::bm) * ((g.N + C::bn - 1) / C::bn);
  constexpr size_t need = C::lds_floats * sizeof(float);
  const bool alone = C::bm * C::bn > 32 * 32 && g.K * (C::bm + C::bn) > kOneBlockWords;
  const size_t bytes = alone && need < kOneBlockLds ? kOneBlockLds : need;
  hipLaunchKernelGGL((gemm_direct_kernel<C, kSplit>), dim3((unsigned)tiles), dim3(C::threads),
                     bytes, s, g.A, g.lda, g.B, g.ldb, g.C, g.ldc, g.M, g.N, g.K);
  return hipGetLastError();
}

// The direct forms, smallest tile last.  ns_per_k: measured time a round of
// 256 tiles (one a CU) takes per unit of K, (t(K = 2048) - t(K = 256)) / 1792.
struct DirectForm {
  int bm, bn, cols;      // tile; columns one load holds (N must reach them)
  double ns_per_k;
  int threads;           // a block's
  hipError_t (*launch)(const GemmProblemF32&, hipStream_t);
  // A row of C holds one load, and the grid counts the call's threads: N of up
  // to 16 takes 4 threads a row in 64 x 16 tiles, 2^32 at 2^30 rows, where the
  // LDS-staged 128-row tiles stay at two a row.
  bool takes(int64_t M, int64_t N) const {
    return N >= cols && launch::grid_fits(((M + bm - 1) / bm) * ((N + bn - 1) / bn), threads);
  }
};
template <bool kSplit, int kFM, int kFN, int kWM, int kWN, int kWK, int kDepth>
constexpr DirectForm direct(double ns_per_k) {
  using C = DirectCfg<kFM, kFN, kWM, kWN, kWK, kDepth>;
  return {C::bm, C::bn, C::fn, ns_per_k, C::threads, launch_direct<C, kSplit>};
}

// A call's time as rounds of 256 tiles, each K steps and the start and end
// of its tiles: measured at K = 64, 2.0 us a round for 64 x 64 and smaller
// tiles, 2.5 for 64 x 128, 3.5 for 128 x 128.
inline double rounds_us(int64_t M, int64_t N, int64_t K, int bm, int bn, double ns_per_k, double ends) {
  const double tiles = (double)((M + bm - 1) / bm) * (double)((N + bn - 1) / bn);
  const double rounds = tiles <= 256 ? 1.0 : (double)(int64_t)((tiles + 255) / 256);
  return rounds * ((double)K * ns_per_k * 1e-3 + ends);
}

// What a round of larger FP32 tiles takes beyond that when there are several:
// measured on 1661 x 2742 to 3001 x 3001 at K = 51, 200 and 801 (64 x 128 at
// K = 200: 14.7 us a round where 9.8 were estimated, and 44 us in three rounds
// against 34 in the LDS-staged tile).  Straight lines between the three K chose
// no better than the steps: over 272 shapes the form taken is 1.2 % slower than
// the fastest either way.
inline double later_rounds_us(int bm, int bn, int64_t K) {
  const int area = bm * bn;
  if (area < 6144) return 0.0;
  if (area == 9216) return K < 100 ? 0.4 : K < 512 ? 1.5 : 0.0;
  if (area < 8192) return K < 100 ? 0.7 : K < 512 ? 2.5 : 1.0;
  return K < 100 ? 2.0 : K < 512 ? 5.0 : 1.0;
}

// The fastest of `count` direct forms by that estimate, or null (*us infinite)
// where none takes the call.
inline const DirectForm* best_direct(const DirectForm* forms, int count, int64_t M, int64_t N,
                                     int64_t K, bool fp32, double* us) {
  const DirectForm* best = nullptr;
  *us = INFINITY;
  for (int i = 0; i < count; ++i) {
    const DirectForm& f = forms[i];
    if (!f.takes(M, N)) continue;
    double ends = 1.5 + f.bm * f.bn / 8192.0;
    if (fp32 && ((M + f.bm - 1) / f.bm) * ((N + f.bn - 1) / f.bn) > 256)
      ends += later_rounds_us(f.bm, f.bn, K);
    const double t = rounds_us(M, N, K, f.bm, f.bn, f.ns_per_k, ends);
    if (t < *us) { best = &f; *us = t; }
  }
  return best;
}

}  // namespace
}  // namespace desc
