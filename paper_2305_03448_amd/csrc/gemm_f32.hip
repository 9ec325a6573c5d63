// gemm_f32.hip -- C = A * B in FP32 on the matrix cores (the "matrix
// multiplication" benchmark of Sec. 5; precision and layout read as FP32,
// row-major, C overwritten).
//
// A is M x K (row stride lda), B is K x N (row stride ldb), C is M x N (row
// stride ldc), all row-major FP32.  Block tiles are BM x BN with a K step of
// BK; the four waves of a block form a 2 x 2 grid, each owning a
// (BM/2) x (BN/2) tile of 32 x 32 v_mfma_f32_32x32x2_f32 fragments.
//
// Per K step, the block copies the A tile into LDS k-major ([BK][BM]) and
// the B tile as it is ([BK][BN]), so that the 64 lanes of a wave read a
// fragment from consecutive LDS words.  The LDS tiles are double buffered:
// the global loads of step t+1 are issued before the matrix ops of step t
// and written to the other buffer after them, one barrier per step.  Edge
// tiles (and unaligned operands) load element by element with zero fill
// and store under guards, so any M, N, K and leading dimensions work.
//
// The tile routine is shared with the grouped GEMM (grouped.hip).
#include "direct_forms.hpp"
#include "gemm_direct.hpp"
#include "gemm_f32.hpp"
#include "launch.hpp"
#include "tuning.hpp"

namespace desc {
namespace {

template <class C, bool kVec>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ A, int64_t lda,
                                                       const float* __restrict__ B, int64_t ldb,
                                                       float* __restrict__ Cm, int64_t ldc,
                                                       int64_t M, int64_t N, int64_t K) {
  __shared__ float lds[gemm_f32::lds_floats<C>()];
  const GemmProblemF32 p{A, lda, B, ldb, Cm, ldc, M, N, K};
  const idx_t tiles_n = (N + C::bn - 1) / C::bn;
  const idx_t t = gemm_f32::xcd_tile(block_x(), (M + C::bm - 1) / C::bm, tiles_n);
  gemm_f32::tile<C, kVec>(p, t / tiles_n, t % tiles_n, lds);
}

template <class C, bool kVec>
__global__ __launch_bounds__(C::threads) __attribute__((amdgpu_waves_per_eu(C::depth)))
void gemm_f32w_kernel(
    const float* __restrict__ A, int64_t lda, const float* __restrict__ B, int64_t ldb,
    float* __restrict__ Cm, int64_t ldc, int64_t M, int64_t N, int64_t K) {
  __shared__ __attribute__((aligned(16))) float lds[C::lds_floats];
  const GemmProblemF32 p{A, lda, B, ldb, Cm, ldc, M, N, K};
  const idx_t tiles_n = (N + C::bn - 1) / C::bn;
  const idx_t t = gemm_f32::xcd_tile(block_x(), (M + C::bm - 1) / C::bm, tiles_n);
  const idx_t tm = t / tiles_n, tn = t % tiles_n;
  if (kVec && gemm_f32::interior_tile<C>(p, tm, tn))
    gemm_f32::tile_rowmajor<C, true, true>(p, tm, tn, lds);
  else
    gemm_f32::tile_rowmajor<C, kVec>(p, tm, tn, lds);
}

// The clamped form (gemm_f32.hpp): tiles inside C, and the ones at its edges.
// It takes 131 registers, three blocks a CU; kBlocks = 4 holds it to 128, at the
// cost of a few spilled words.
template <class C, int kBlocks>
__global__ __launch_bounds__(C::threads) __attribute__((amdgpu_waves_per_eu(kBlocks)))
void gemm_f32c_kernel(
    const float* __restrict__ A, int64_t lda, const float* __restrict__ B, int64_t ldb,
    float* __restrict__ Cm, int64_t ldc, int64_t M, int64_t N, int64_t K) {
  __shared__ __attribute__((aligned(16))) float lds[C::lds_floats];
  const GemmProblemF32 p{A, lda, B, ldb, Cm, ldc, M, N, K};
  const auto t = layout::xcd_run_tile(block_x().index(), (M + C::bm - 1) / C::bm,
                                      (N + C::bn - 1) / C::bn);
  if ((t.m + 1) * C::bm <= M && (t.n + 1) * C::bn <= N)
    gemm_f32::tile_rowmajor<C, true, true, true>(p, t.m, t.n, lds);
  else
    gemm_f32::tile_rowmajor<C, true, false, true>(p, t.m, t.n, lds);
}

template <class C>
hipError_t launch_gemm_w(const float* A, int64_t lda, const float* B, int64_t ldb, float* Cm,
                         int64_t ldc, int64_t M, int64_t N, int64_t K, hipStream_t s) {
  const int64_t tiles = ((M + C::bm - 1) / C::bm) * ((N + C::bn - 1) / C::bn);
  // the clamped group loads need K and N in whole groups of four (K, N >= 4)
  if (gemm_f32::vec_ok(A, lda, B, ldb) && K % 4 == 0 && N % 4 == 0 && K > 0)
    hipLaunchKernelGGL((gemm_f32w_kernel<C, true>), dim3((unsigned)tiles), dim3(C::threads), 0,
                       s, A, lda, B, ldb, Cm, ldc, M, N, K);
  else
    hipLaunchKernelGGL((gemm_f32w_kernel<C, false>), dim3((unsigned)tiles), dim3(C::threads), 0,
                       s, A, lda, B, ldb, Cm, ldc, M, N, K);
  return hipGetLastError();
}

// The clamped form where the call's spans allow it, else the guarded one.
// 769 to 1024 tiles are one residency of four blocks a CU and leave three a
// nearly empty last round: 4000 x 4000 at K = 512 156 us in three (140 in the
// guarded form), 129 in four; 2796 x 5424 x 1012 294 and 247; about even where the
// rounds happen to fit (2496 x 5760 x 896 218 / 216); 3 % the other way below
// K = 100 (6272 x 2368 x 96 32.7 / 33.7), and up to 18 % past 1024 tiles.
template <class C>
hipError_t launch_gemm_c(const GemmProblemF32& g, hipStream_t s) {
  if (!gemm_f32::clamped_tile<C>(g))
    return launch_gemm_w<C>(g.A, g.lda, g.B, g.ldb, g.C, g.ldc, g.M, g.N, g.K, s);
  const int64_t tiles = ((g.M + C::bm - 1) / C::bm) * ((g.N + C::bn - 1) / C::bn);
  if (tiles > 3 * 256 && tiles <= 4 * 256 && g.K >= 128)
    hipLaunchKernelGGL((gemm_f32c_kernel<C, 4>), dim3((unsigned)tiles), dim3(C::threads), 0, s,
                       g.A, g.lda, g.B, g.ldb, g.C, g.ldc, g.M, g.N, g.K);
  else
    hipLaunchKernelGGL((gemm_f32c_kernel<C, C::depth>), dim3((unsigned)tiles), dim3(C::threads), 0,
                       s, g.A, g.lda, g.B, g.ldb, g.C, g.ldc, g.M, g.N, g.K);
  return hipGetLastError();
}

template <class C>
hipError_t launch_gemm(const float* A, int64_t lda, const float* B, int64_t ldb, float* Cm,
                       int64_t ldc, int64_t M, int64_t N, int64_t K, hipStream_t s) {
  const int64_t tiles = ((M + C::bm - 1) / C::bm) * ((N + C::bn - 1) / C::bn);
  const bool vec = gemm_f32::vec_ok(A, lda, B, ldb);
  if (vec)
    hipLaunchKernelGGL((gemm_f32_kernel<C, true>), dim3((unsigned)tiles), dim3(256), 0, s, A, lda,
                       B, ldb, Cm, ldc, M, N, K);
  else
    hipLaunchKernelGGL((gemm_f32_kernel<C, false>), dim3((unsigned)tiles), dim3(256), 0, s, A,
                       lda, B, ldb, Cm, ldc, M, N, K);
  return hipGetLastError();
}

// The FP32 direct forms.  The matrix work of a 128 x 128 tile alone is 53 ns;
// small tiles pay for their loads instead (16 x 16: 2.2 ns for 0.8 ns of
// matrix work), but a shape with few tiles is faster in more, smaller ones.
constexpr DirectForm kDirect[] = {
    direct<false, 4, 4, 2, 2, 1, 3>(67.1),   // 128 x 128
    direct<false, 4, 4, 1, 2, 2, 2>(36.6),   // 64 x 128
    direct<false, 4, 4, 2, 1, 2, 2>(38.3),   // 128 x 64
    direct<false, 3, 3, 2, 2, 1, 3>(42.6),   // 96 x 96
    direct<false, 4, 3, 1, 2, 2, 3>(27.6),   // 64 x 96
    direct<false, 3, 4, 2, 1, 2, 3>(27.7),   // 96 x 64
    direct<false, 4, 4, 1, 1, 4, 2>(18.8),   // 64 x 64
    direct<false, 3, 4, 1, 1, 4, 4>(13.5),   // 48 x 64
    direct<false, 4, 3, 1, 1, 4, 4>(13.6),   // 64 x 48
    direct<false, 3, 3, 1, 1, 4, 4>(10.4),   // 48 x 48
    direct<false, 2, 4, 1, 1, 4, 4>(9.0),    // 32 x 64
    direct<false, 4, 2, 1, 1, 4, 4>(10.7),   // 64 x 32
    direct<false, 2, 2, 1, 1, 4, 6>(5.8),    // 32 x 32
    direct<false, 1, 4, 1, 1, 4, 4>(4.9),    // 16 x 64
    direct<false, 4, 1, 1, 1, 4, 4>(8.4),    // 64 x 16
    direct<false, 1, 2, 1, 1, 8, 6>(4.1),    // 16 x 32
    direct<false, 2, 1, 1, 1, 8, 6>(4.8),    // 32 x 16
    direct<false, 1, 1, 1, 1, 16, 4>(2.2),   // 16 x 16
};
constexpr int kDirectForms = (int)(sizeof(kDirect) / sizeof(kDirect[0]));

// Short K over many tiles is bound by C and by the ends of the tiles, which
// three LDS-staged 64 x 64 blocks a CU overlap and the direct forms, alone on
// a CU or two to it, do not: 102400 x 64 x 32 11.9 us against 18.4, 204800 x 32 x 16
// 14.7 / 19.5, 20000 x 256 x 64 13.3 / 15.4, 3200 x 512 x 16 4.8 / 5.6.  The
// staged form's time by tiles of 64 x 64 (t) and K: 400 tiles 4.8 us at K = 16 and
// 7.1 at 64, 3200 tiles 14.4 and 26; direct forms take 2.5 us more than
// their estimate, which counts rounds alone, up to one residency of the staged
// form (768 tiles) and 2 beyond.  Not where the direct form runs one round of
// tiles that the other would need two for (25600 x 100 x 16 5.6 / 7.1), not for
// narrow C, of which a 64-wide tile wastes most (102400 x 16 x 64 9.7 / 15.8), and on
// operands that are not in 16-byte groups, which the staged form reads word by
// word, only up to K = 16 (204800 x 30: K = 16 15.3 / 19.7, 32 22.0 / 23.5, 64 35.7 / 26.0).
bool short_k_staged(const GemmProblemF32& g, const DirectForm& d, double direct_us) {
  const int64_t t = ((g.M + 63) / 64) * ((g.N + 63) / 64);
  const int64_t direct_tiles = ((g.M + d.bm - 1) / d.bm) * ((g.N + d.bn - 1) / d.bn);
  const bool vec = gemm_f32::vec_ok(g.A, g.lda, g.B, g.ldb);
  if (g.N < 24 || g.K > (!vec ? 16 : g.N < 48 ? 32 : 64) || g.M * g.N * g.K >= (int64_t)1 << 30)
    return false;
  if (t <= 256 || (t > 768 && direct_tiles <= 256)) return false;
  const double r = (double)t / 256, first = r < 3 ? r : 3.0, k = (double)g.K * 1e-3;
  return 3.3 + 12.2 * k * first + r * (0.7 + 14.9 * k) < direct_us + (t <= 768 ? 2.5 : 2.0);
}

// "_rm": the row-major-A tile form; "_w8": eight waves (2 x 4).  "by_shape":
// a direct form or the LDS-staged 128 x 128 tile, whichever the call's M, N
// and K make faster; "dBMxBN": that direct form (by_shape where a row of C is
// shorter than one load, or a stride is beyond the direct forms').
constexpr const char* kNames[] = {"m128n128k16", "m256n128k16", "m128n128k32", "m64n64k16",
                                  "m256n256k16_rm_w8_d2", "m256n128k16_rm", "m256n128k16_rm_d2",
                                  "m128n128k16_rm", "m128n128k16_rm_d2", "m128n128k16_rm_d2_x16",
                                  "m256n128k16_rm_d2_x16", "by_shape",
                                  "d128x128", "d64x128", "d128x64", "d96x96", "d64x96", "d96x64",
                                  "d64x64", "d48x64", "d64x48", "d48x48", "d32x64", "d64x32",
                                  "d32x32", "d16x64", "d64x16", "d16x32", "d32x16", "d16x16",
                                  "m128n128k16_c"};
constexpr int kByShape = 11, kCount = (int)(sizeof(kNames) / sizeof(kNames[0]));
constexpr int kClamped = kByShape + 1 + kDirectForms;   // the clamped 128 x 128 form
static_assert(kCount == kClamped + 1, "one name per configuration");
using Staged = gemm_f32::GemmCfgF32W<128, 128, 16, 2, 2, 2, true>;
constexpr int kDefaults[tune::kClasses] = {kByShape, kByShape, kByShape, kByShape};
const bool kRegistered =
    (tune::register_op(tune::kGemmF32, "gemm_f32", kCount, kNames, kDefaults), true);

}  // namespace

namespace launch {

hipError_t gemm_f32(const float* A, int64_t lda, const float* B, int64_t ldb, float* Cm,
                    int64_t ldc, int64_t M, int64_t N, int64_t K, hipStream_t s) {
  if (M == 0 || N == 0) return hipSuccess;
  (void)kRegistered;
  const int cls = tune::size_class(tune::kGemmF32, M * N * (K ? K : 1));
  int cfg = tune::get(tune::kGemmF32, cls);
  const GemmProblemF32 g{A, lda, B, ldb, Cm, ldc, M, N, K};
  if (cfg == kClamped) return launch_gemm_c<Staged>(g, s);
  if (cfg >= kByShape) {
    const bool strides = lda <= kDirectMaxLd && ldb <= kDirectMaxLd;
    if (cfg > kByShape && strides && kDirect[cfg - kByShape - 1].takes(M, N))
      return kDirect[cfg - kByShape - 1].launch(g, s);
    // The LDS-staged 128 x 128 tile, up to three blocks a CU, is the faster
    // one per unit of K once several rounds of its tiles run: 67 ns a round
    // of 256 tiles for one round, 63 for two, 58-60 from four on, and 2 us of
    // ends, 4 at short K (4096^3: 941 us against 1044 in direct tiles; 8192 x 8192 x 64: 94
    // against 115; but 1536 x 3072 x 2048, whose 288 tiles leave a second
    // round nearly empty: 260 against 171 us in 96 x 64 direct tiles).
    if (strides) {
      double us = 0;
      const DirectForm* d = best_direct(kDirect, kDirectForms, M, N, K, true, &us);
      const double tiles = (double)((M + 127) / 128) * (double)((N + 127) / 128);
      const double ns = 58.0 + 9.0 / (tiles <= 256 ? 1.0 : tiles / 256);
      const bool staged_ok = gemm_f32::clamped_tile<Staged>(g);
      if (d && (!staged_ok || us <= rounds_us(M, N, K, 128, 128, ns, K < 512 ? 4.0 : 2.0)))
        return short_k_staged(g, *d, us)
                   ? launch_gemm<GemmCfgF32<64, 64, 16>>(A, lda, B, ldb, Cm, ldc, M, N, K, s)
                   : d->launch(g, s);
    }
    // whole tiles of aligned rows keep the form without clamps (4096^3: 941
    // against 956 us)
    if (!gemm_f32::vec_ok(A, lda, B, ldb) || M % 128 != 0 || N % 128 != 0 || K % 16 != 0)
      return launch_gemm_c<Staged>(g, s);
    cfg = 9;
  }
  switch (cfg) {
    case 1: return launch_gemm<GemmCfgF32<256, 128, 16>>(A, lda, B, ldb, Cm, ldc, M, N, K, s);
    case 2: return launch_gemm<GemmCfgF32<128, 128, 32>>(A, lda, B, ldb, Cm, ldc, M, N, K, s);
    case 3: return launch_gemm<GemmCfgF32<64, 64, 16>>(A, lda, B, ldb, Cm, ldc, M, N, K, s);
    case 4:
      return launch_gemm_w<gemm_f32::GemmCfgF32W<256, 256, 16, 2, 4, 2>>(A, lda, B, ldb, Cm, ldc, M, N, K, s);
    case 5:
      return launch_gemm_w<gemm_f32::GemmCfgF32W<256, 128, 16, 2, 2>>(A, lda, B, ldb, Cm, ldc, M, N, K, s);
    case 6:
      return launch_gemm_w<gemm_f32::GemmCfgF32W<256, 128, 16, 2, 2, 2>>(A, lda, B, ldb, Cm, ldc, M, N, K, s);
    case 7:
      return launch_gemm_w<gemm_f32::GemmCfgF32W<128, 128, 16, 2, 2>>(A, lda, B, ldb, Cm, ldc, M, N, K, s);
    case 8:
      return launch_gemm_w<gemm_f32::GemmCfgF32W<128, 128, 16, 2, 2, 2>>(A, lda, B, ldb, Cm, ldc, M, N, K, s);
    case 9:
      return launch_gemm_w<gemm_f32::GemmCfgF32W<128, 128, 16, 2, 2, 2, true>>(A, lda, B, ldb, Cm, ldc, M, N, K, s);
    case 10:
      return launch_gemm_w<gemm_f32::GemmCfgF32W<256, 128, 16, 2, 2, 2, true>>(A, lda, B, ldb, Cm, ldc, M, N, K, s);
    default: return launch_gemm<GemmCfgF32<128, 128, 16>>(A, lda, B, ldb, Cm, ldc, M, N, K, s);
  }
}

}  // namespace launch
}  // namespace desc
