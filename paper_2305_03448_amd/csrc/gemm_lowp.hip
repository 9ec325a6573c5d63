// gemm_lowp.hip -- the precision forms of C = A * B: three-product split
// bfloat16 with FP32 accumulation, and e4m3 with per-row / per-column
// absmax scaling.  Large products prepare their operands in the workspace and
// run direct-to-LDS tiles (gemm_dma.hpp) or the NT tile of gemm_nt.hpp over
// them; small ones take the FP32 operands or, in FP8, direct tiles over the
// codes (gemm_direct.hpp, gemm_fp8_fused.hpp, gemm_direct_nt.hpp).
//
// BF16x3.  a = hi + lo with hi = bf16(a), lo = bf16(a - hi) (a - hi is exact
// in FP32), likewise for b; C ~ Ah*Bh + Ah*Bl + Al*Bh (the Al*Bl term is
// below FP32 resolution).  Pre-pass: A -> Ah, Al as [Mp][Kp] bf16 (an
// element-wise pass), B -> Bh^T, Bl^T as [Np][Kp] bf16 (an LDS-tiled
// transpose, split on the way); for the direct-to-LDS tiles one launch and one
// plane per operand (split_paired_kernel); the fused and the direct forms take
// the FP32 operands.
//
// FP8.  alpha_i = max_k |a_ik|; q_ik = e4m3(a_ik * (448 / alpha_i)) with one
// FP32 division and one FP32 multiply; s_i = alpha_i / 448 (an all-zero row
// uses 448/alpha = 1 and s = 0).  Columns of B likewise with beta_j.  Then
// C_ij = s_i * t_j * sum_k q_ik q_kj, the sum on the matrix cores in FP32.
// Pre-pass, two launches: one block per row of A (absmax, then encode)
// beside the column absmax of B as partial maxima over K slices; then a pass
// over B that encodes with the column scales and writes q^T as [Np][Kp].  Up
// to K = 2048 one launch does both (fp8_once_kernel), but for a wide B of
// short K (wide_b).
//
// Padding: Mp, Np are multiples of 256 and Kp a multiple of 128 elements;
// the pre-pass writes zeros there, so the GEMM main loop has no guards.
#include <algorithm>
#include <cmath>

#include "common.hpp"
#include "direct_forms.hpp"
#include "gemm_direct_nt.hpp"
#include "gemm_dma.hpp"
#include "gemm_fp8_fused.hpp"
#include "gemm_nt.hpp"
#include "launch.hpp"
#include "lowp.hpp"
#include "tuning.hpp"
#include "view.hpp"
#include "wave.hpp"

namespace desc {
namespace {

constexpr int kBlock = 256;
constexpr int64_t kPadMN = 256, kPadK = 128;

int64_t round_up(int64_t v, int64_t m) { return (v + m - 1) / m * m; }
size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// ------------------------------------------------------------------ split
typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
typedef uint8_t u8x4 __attribute__((ext_vector_type(4)));

// Rows of A (M x K, stride lda) -> hi, lo (rows_out x k_out, stride ldh);
// positions beyond M or K are written as zero.  Thread = 4 consecutive k:
// one 16-byte load and two 8-byte stores when the group is whole and
// aligned (vec_in: A and lda allow float4; vec_out: hi, lo and ldh allow
// 8-byte stores), element by element otherwise.
__global__ __launch_bounds__(kBlock) void split_rows_kernel(const float* __restrict__ A,
                                                            int64_t M, int64_t K, int64_t lda,
                                                            uint16_t* __restrict__ hi,
                                                            uint16_t* __restrict__ lo,
                                                            int64_t rows_out, int64_t k_out,
                                                            int64_t ldh, bool vec_in,
                                                            bool vec_out) {
  auto block = block_x();
  auto thread = thread_x<kBlock>();
  auto a = matrix(A, M, lda);
  auto h = matrix(hi, rows_out, ldh);
  auto l = matrix(lo, rows_out, ldh);
  const int64_t groups = (k_out + 3) / 4;
  const int64_t total = rows_out * groups;
  for (idx_t g = block.index() * kBlock + thread.index(); g < total;
       g += block.count() * kBlock) {
    const idx_t r = g / groups, c = 4 * (g % groups);
    f32x4 v;
    if (vec_in && r < M && c + 4 <= K) {
      v = *(const f32x4*)&a.at(r, c);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = (r < M && c + j < K) ? a.at(r, c + j) : 0.f;
    }
    const lowp::Split4 sp = lowp::split_bf16x4(v[0], v[1], v[2], v[3]);
    const u16x4 vh = sp.hi, vl = sp.lo;
    if (vec_out && c + 4 <= k_out) {
      *(u16x4*)&h.at(r, c) = vh;
      *(u16x4*)&l.at(r, c) = vl;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (c + j < k_out) {
          h.at(r, c + j) = vh[j];
          l.at(r, c + j) = vl[j];
        }
    }
  }
}

// Columns of B (K x N, stride ldb) -> hi^T, lo^T (n_out x k_out, stride ldh).
// 64 x 64 tiles of B through LDS; grid (k tiles, n tiles).  Reads run along
// n (thread = 4 columns of one row), writes along k (thread = 4 consecutive
// k of one output row, two 8-byte stores).
__global__ __launch_bounds__(kBlock) void split_cols_t_kernel(const float* __restrict__ B,
                                                              int64_t K, int64_t N, int64_t ldb,
                                                              uint16_t* __restrict__ hi,
                                                              uint16_t* __restrict__ lo,
                                                              int64_t n_out, int64_t k_out,
                                                              int64_t ldh, bool vec_in,
                                                              bool vec_out) {
  __shared__ float lds[64 * 65];
  auto kt = block_x();
  auto nt = block_y();
  auto thread = thread_x<kBlock>();
  auto tile = matrix(lds, 64, 65);
  auto b = matrix(B, K, ldb);
  auto h = matrix(hi, n_out, ldh);
  auto l = matrix(lo, n_out, ldh);
  const idx_t k0 = kt.index() * 64, n0 = nt.index() * 64;
  const int tx = (int)thread.index() % 16, ty = (int)thread.index() / 16;
#pragma unroll
  for (int i = 0; i < 4; ++i) {                 // rows ty + 16 i, columns 4 tx ..
    const idx_t r = ty + 16 * i, c = 4 * tx;
    f32x4 v;
    if (vec_in && k0 + r < K && n0 + c + 4 <= N) {
      v = *(const f32x4*)&b.at(k0 + r, n0 + c);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        v[j] = (k0 + r < K && n0 + c + j < N) ? b.at(k0 + r, n0 + c + j) : 0.f;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) tile.at(r, c + j) = v[j];
  }
  sync(thread);
#pragma unroll
  for (int i = 0; i < 4; ++i) {                 // output rows (columns of B) ty + 16 i
    const idx_t c = ty + 16 * i, r = 4 * tx;
    if (n0 + c >= n_out) continue;
    const lowp::Split4 sp = lowp::split_bf16x4(tile.at(r, c), tile.at(r + 1, c),
                                               tile.at(r + 2, c), tile.at(r + 3, c));
    const u16x4 vh = sp.hi, vl = sp.lo;
    if (vec_out && k0 + r + 4 <= k_out) {
      *(u16x4*)&h.at(n0 + c, k0 + r) = vh;
      *(u16x4*)&l.at(n0 + c, k0 + r) = vl;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (k0 + r + j < k_out) {
          h.at(n0 + c, k0 + r + j) = vh[j];
          l.at(n0 + c, k0 + r + j) = vl[j];
        }
    }
  }
}

// ------------------------------------------------------------------ e4m3
__device__ __forceinline__ float block_max(float v, float* red) {
  auto thread = thread_x<kBlock>();
  auto wv = wave_of_block<kBlock>();
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) v = fmaxf(v, __shfl_xor(v, s, 64));
  if (lane_of_wave().index() == 0) red[wv.index()] = v;
  sync(thread);
  float m = red[0];
#pragma unroll
  for (int w = 1; w < kBlock / kWave; ++w) m = fmaxf(m, red[w]);
  return m;
}

// One block per output row: absmax over the row, then encode, 4 consecutive
// k per thread (16-byte loads and 4-byte stores when whole and aligned).
// Rows of up to kRowCache * 1024 elements stay in registers between the two
// phases, so the row is read once; longer rows are read again to encode.
// q is rows_out x k_out (stride ldq); rows >= M and columns >= K get zero.
constexpr int kRowCache = 8;   // float4 per thread

// Row r of rows_out (the block's row; the caller's grid may hold other work).
// kNt: a cached row is read non-temporally.
template <bool kNt>
__device__ __forceinline__ void quant_row(const float* __restrict__ A, int64_t M, int64_t K,
                                          int64_t lda, uint8_t* __restrict__ q, int64_t rows_out,
                                          int64_t k_out, int64_t ldq, float* __restrict__ scale,
                                          bool vec_in, bool vec_out, idx_t r) {
  __shared__ float red[kBlock / kWave];
  auto thread = thread_x<kBlock>();
  auto a = matrix(A, M, lda);
  auto qr = matrix(q, rows_out, ldq).idx(r);
  auto load4 = [&](idx_t c) {
    f32x4 v;
    if (vec_in && r < M && c + 4 <= K) {
      v = *(const f32x4*)&a.at(r, c);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = (r < M && c + j < K) ? a.at(r, c + j) : 0.f;
    }
    return v;
  };
  auto encode = [&](idx_t c, const f32x4& v, float inv) {
    // positions past the row (padding) get code 0
    uint32_t keep = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) keep |= (r < M && c + j < K) ? (0xffu << (8 * j)) : 0u;
    const uint32_t w = lowp::e4m3x4(v[0] * inv, v[1] * inv, v[2] * inv, v[3] * inv) & keep;
    const u8x4 e = __builtin_bit_cast(u8x4, w);
    if (vec_out && c + 4 <= k_out) {
      *(u8x4*)&qr[c] = e;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (c + j < k_out) qr[c + j] = e[j];
    }
  };
  const bool cached = k_out <= 4 * kBlock * kRowCache && K <= k_out;
  float amax = 0.f;
  f32x4 cache[kRowCache];
  if (cached && vec_in && r < M && K % 4 == 0) {
    // Branch-free: every load reads a valid address (column 0 past the end
    // of the row) and the value is dropped by a select, so the loads are all
    // in flight together instead of one conditional load after another.
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < kRowCache; ++i) {
      const idx_t c = 4 * (thread.index() + kBlock * i);
      const f32x4* p = (const f32x4*)&a.at(r, c < K ? c : 0);
      f32x4 v;
      if constexpr (kNt) v = __builtin_nontemporal_load(p);
      else v = *p;
      cache[i] = c < K ? v : zero;
    }
#pragma unroll
    for (int i = 0; i < kRowCache; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) amax = fmaxf(amax, fabsf(cache[i][j]));
  } else if (cached) {
#pragma unroll
    for (int i = 0; i < kRowCache; ++i) {
      const idx_t c = 4 * (thread.index() + kBlock * i);
      cache[i] = c < K ? load4(c) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < 4; ++j) amax = fmaxf(amax, fabsf(cache[i][j]));
    }
  } else {
    for (idx_t c = 4 * thread.index(); c < K; c += 4 * kBlock) {
      const f32x4 v = load4(c);
#pragma unroll
      for (int j = 0; j < 4; ++j) amax = fmaxf(amax, fabsf(v[j]));
    }
  }
  amax = block_max(amax, red);
  const float inv = amax > 0.f ? 448.0f / amax : 1.0f;
  if (cached) {
#pragma unroll
    for (int i = 0; i < kRowCache; ++i) {
      const idx_t c = 4 * (thread.index() + kBlock * i);
      if (c < k_out) encode(c, cache[i], inv);
    }
  } else {
    for (idx_t c = 4 * thread.index(); c < k_out; c += 4 * kBlock) encode(c, load4(c), inv);
  }
  if (thread.index() == 0) array(scale, rows_out)[r] = amax / 448.0f;
}

__global__ __launch_bounds__(kBlock) void quant_rows_kernel(const float* __restrict__ A,
                                                            int64_t M, int64_t K, int64_t lda,
                                                            uint8_t* __restrict__ q,
                                                            int64_t k_out, int64_t ldq,
                                                            float* __restrict__ scale,
                                                            bool vec_in, bool vec_out) {
  auto row = block_x();
  quant_row<false>(A, M, K, lda, q, row.count(), k_out, ldq, scale, vec_in, vec_out, row.index());
}

// Partial column maxima of |B| over K slices: part[s][n] for slice s of
// `rows_per` rows; grid (column blocks of 1024, slices).  Thread = 4
// consecutive columns, read as one 16-byte vector per row when aligned;
// eight rows are loaded before they are combined.
// Column block cb (kBlock * 4 columns) of slice sl (of nslices).
__device__ __forceinline__ void colmax_part(const float* __restrict__ B, int64_t K, int64_t N,
                                            int64_t ldb, int64_t rows_per,
                                            float* __restrict__ part, int64_t ldp, bool vec_in,
                                            idx_t cb, idx_t sl, idx_t nslices) {
  auto thread = thread_x<kBlock>();
  auto b = matrix(B, K, ldb);
  const idx_t n = (cb * kBlock + thread.index()) * 4;
  const idx_t k0 = sl * rows_per;
  const idx_t k1 = k0 + rows_per < K ? k0 + rows_per : K;
  f32x4 m = {0.f, 0.f, 0.f, 0.f};
  if (vec_in && n + 4 <= N) {
#pragma unroll 8
    for (idx_t k = k0; k < k1; ++k) {
      const f32x4 v = *(const f32x4*)&b.at(k, n);
#pragma unroll
      for (int j = 0; j < 4; ++j) m[j] = fmaxf(m[j], fabsf(v[j]));
    }
  } else {
    for (idx_t k = k0; k < k1; ++k)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (n + j < N) m[j] = fmaxf(m[j], fabsf(b.at(k, n + j)));
  }
  auto pr = matrix(part, nslices, ldp).idx(sl);
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (n + j < ldp) pr[n + j] = m[j];
}

__global__ __launch_bounds__(kBlock) void colmax_partial_kernel(const float* __restrict__ B,
                                                                int64_t K, int64_t N,
                                                                int64_t ldb, int64_t rows_per,
                                                                float* __restrict__ part,
                                                                int64_t ldp, bool vec_in) {
  auto sl = block_y();
  colmax_part(B, K, N, ldb, rows_per, part, ldp, vec_in, block_x().index(), sl.index(),
              sl.count());
}

// The FP8 GEMM's first pass in one launch: the column-maximum partials of B
// (the first cblocks * nslices blocks, the longer ones, so they start first)
// and the row quantisation of A (one block per padded row), which do not
// depend on each other.
template <bool kNt>
__global__ __launch_bounds__(kBlock) void fp8_prepass_kernel(
    const float* __restrict__ A, int64_t M, int64_t K, int64_t lda, uint8_t* __restrict__ qa,
    int64_t rows_out, int64_t k_out, int64_t ldqa, float* __restrict__ sa, bool a_vec_in,
    const float* __restrict__ B, int64_t N, int64_t ldb, int64_t rows_per,
    float* __restrict__ part, int64_t ldp, bool b_vec_in, int64_t cblocks, int64_t nslices) {
  const idx_t blk = block_x().index(), col_blocks = cblocks * nslices;
  if (blk < col_blocks)
    colmax_part(B, K, N, ldb, rows_per, part, ldp, b_vec_in, blk % cblocks, blk / cblocks,
                nslices);
  else
    quant_row<kNt>(A, M, K, lda, qa, rows_out, k_out, ldqa, sa, a_vec_in, true, blk - col_blocks);
}

// Encode tiles of 64 k x 64 columns of B with their column scales and
// write them transposed: qt is n_out x k_out (stride ldq).  A block
// takes one k tile of one column block; the first block of each column
// block also writes the column scales.  The tile's loads are issued before
// the column maxima are gathered from the slice partials, so the two sets
// of loads are in flight together.  Reads run along n (thread = 4 columns
// of one row), writes along k (thread = 4 consecutive k, one 4-byte store).
__global__ __launch_bounds__(kBlock) void quant_cols_tile_kernel(const float* __restrict__ B,
                                                                 int64_t K, int64_t N, int64_t ldb,
                                                                 const float* __restrict__ part,
                                                                 int64_t nslices, int64_t ldp,
                                                                 uint8_t* __restrict__ qt,
                                                                 int64_t n_out, int64_t k_out,
                                                                 int64_t ldq,
                                                                 float* __restrict__ scale,
                                                                 bool vec_in, bool vec_out) {
  constexpr int kKT = 64;
  constexpr int kRows = kKT / 16;               // rows of the tile per thread
  constexpr int kLanesPerRow = kKT / 4;         // threads per output row
  constexpr int kOutRows = kBlock / kLanesPerRow;
  __shared__ uint8_t codes[kKT * 68];
  __shared__ float inv_s[64];
  __shared__ float pmax[4][64];
  auto kt = block_x();
  auto nt = block_y();
  auto thread = thread_x<kBlock>();
  auto tile = matrix(codes, kKT, 68);
  auto b = matrix(B, K, ldb);
  auto pm = matrix(part, nslices, ldp);
  auto out = matrix(qt, n_out, ldq);
  const idx_t n0 = nt.index() * 64, k0 = kt.index() * kKT;
  const int tx = (int)thread.index() % 16, ty = (int)thread.index() / 16;
  f32x4 v[kRows];
#pragma unroll
  for (int i = 0; i < kRows; ++i) {             // rows ty + 16 i, columns 4 tx ..
    const idx_t r = ty + 16 * i, c = 4 * tx;
    if (vec_in && k0 + r < K && n0 + c + 4 <= N) {
      v[i] = *(const f32x4*)&b.at(k0 + r, n0 + c);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        v[i][j] = (k0 + r < K && n0 + c + j < N) ? b.at(k0 + r, n0 + c + j) : 0.f;
    }
  }
  {
    // column maxima of the 64 columns from the slice partials: thread
    // (g, c) takes slices g, g + 4, ... of column c (loads coalesced along
    // the columns, independent, so they are in flight together)
    const int c = (int)thread.index() % 64, g = (int)thread.index() / 64;
    const idx_t n = n0 + c;
    float m = 0.f;
    if (n < N)
#pragma unroll 8
      for (idx_t sl = g; sl < nslices; sl += 4) m = fmaxf(m, pm.at(sl, n));
    pmax[g][c] = m;
  }
  sync(thread);
  if (thread.index() < 64) {
    const int c = (int)thread.index();
    const idx_t n = n0 + c;
    const float m = fmaxf(fmaxf(pmax[0][c], pmax[1][c]), fmaxf(pmax[2][c], pmax[3][c]));
    inv_s[c] = m > 0.f ? 448.0f / m : 1.0f;
    if (kt.index() == 0 && n < n_out) array(scale, n_out)[n] = m / 448.0f;
  }
  sync(thread);
#pragma unroll
  for (int i = 0; i < kRows; ++i) {
    const idx_t r = ty + 16 * i, c = 4 * tx;
    uint32_t keep = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) keep |= (k0 + r < K && n0 + c + j < N) ? (0xffu << (8 * j)) : 0u;
    const uint32_t w = lowp::e4m3x4(v[i][0] * inv_s[c], v[i][1] * inv_s[c + 1],
                                    v[i][2] * inv_s[c + 2], v[i][3] * inv_s[c + 3]) & keep;
    *(u8x4*)&tile.at(r, c) = __builtin_bit_cast(u8x4, w);
  }
  sync(thread);
  const int ox = (int)thread.index() % kLanesPerRow, oy = (int)thread.index() / kLanesPerRow;
#pragma unroll
  for (int i = 0; i < 64 / kOutRows; ++i) {     // output rows oy + kOutRows i, k = 4 ox ..
    const idx_t c = oy + kOutRows * i, r = 4 * ox;
    if (n0 + c >= n_out) continue;
    u8x4 e;
#pragma unroll
    for (int j = 0; j < 4; ++j) e[j] = tile.at(r + j, c);
    if (vec_out && k0 + r + 4 <= k_out) {
      *(u8x4*)&out.at(n0 + c, k0 + r) = e;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (k0 + r + j < k_out) out.at(n0 + c, k0 + r + j) = e[j];
    }
  }
}

// The same encode of large matrices and of unaligned ones.  A thread holds 16 consecutive k of four columns, so it stores
// 16 codes of a column at once and nothing passes through LDS; a wave is 128 k
// x 32 columns, whole 128-byte lines on both sides; kW of a block's four waves
// lie along k, the others along the columns.  The values are loaded before the
// column maxima are gathered from the slice partials, so the two sets of loads
// are in flight together; the first block of each column block also writes the
// column scales.  Bound by memory: 8192 x 8192 60 us where tiles of 128 k
// through LDS took 70.
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));   // any element alignment
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(1)));
constexpr int kEncodeRows = 16;   // k per thread

// Rows k .. k + kR of columns n .. n + 3 of B, zero outside it.  `whole`: every
// column is inside; rows past K then read the last one and are dropped, so that
// every load is unconditional.
template <int kR, bool kNt>
__device__ __forceinline__ void load_cols(const float* __restrict__ B, int64_t K, int64_t N,
                                          int64_t ldb, idx_t k, idx_t n, bool whole,
                                          f32x4 (&v)[kR]) {
  auto b = matrix(B, K, ldb);
  if (whole) {
#pragma unroll
    for (int j = 0; j < kR; ++j) {
      const f32x4_any* p = (const f32x4_any*)&b.at(k + j < K ? k + j : K - 1, n);
      if constexpr (kNt) v[j] = __builtin_nontemporal_load(p);
      else v[j] = *p;
    }
#pragma unroll
    for (int j = 0; j < kR; ++j)
      if (k + j >= K) v[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  } else {
#pragma unroll
    for (int j = 0; j < kR; ++j)
#pragma unroll
      for (int c = 0; c < 4; ++c) v[j][c] = k + j < K && n + c < N ? b.at(k + j, n + c) : 0.f;
  }
}

// The byte mask of the first n of four codes.
__device__ __forceinline__ uint32_t code_mask(int64_t n) {
  return n >= 4 ? ~0u : n <= 0 ? 0u : (1u << (8 * (int)n)) - 1u;
}

// The codes of column c of v, the first `valid` of them kept, the others 0.
template <int kR>
__device__ __forceinline__ auto encode_col(const f32x4 (&v)[kR], int c, float inv, int64_t valid) {
  typedef uint32_t Codes __attribute__((ext_vector_type(kR / 4)));
  Codes e;
#pragma unroll
  for (int d = 0; d < kR / 4; ++d)
    e[d] = lowp::e4m3x4(v[4 * d][c] * inv, v[4 * d + 1][c] * inv, v[4 * d + 2][c] * inv,
                        v[4 * d + 3][c] * inv) &
           code_mask(valid - 4 * d);
  return e;
}

// The split-BF16 pre-pass of the direct-to-LDS tiles, one launch: blocks of 512
// k x 32 columns of B as above, then blocks of 2048 groups of 4 consecutive k
// of A.  Both write rows that hold, for every 32 k, 32 hi and then 32 lo
// values: whole lines.  Bound by memory: 43 us at 4096 x 4096 x 4096 (268
// MB) where the two launches above take 22 and 28.
constexpr int kPairGroups = 8;   // groups of A per thread

// 8 values, hi and lo, at group g (of 8 k) of a paired row.
__device__ __forceinline__ void store_pair(u32x4* row, idx_t g, const float (&v)[8]) {
  const lowp::Split4 x = lowp::split_bf16x4(v[0], v[1], v[2], v[3]);
  const lowp::Split4 y = lowp::split_bf16x4(v[4], v[5], v[6], v[7]);
  const auto join = [](lowp::bf16x4_bits p, lowp::bf16x4_bits q) {
    const lowp::u32x2_bits a = __builtin_bit_cast(lowp::u32x2_bits, p);
    const lowp::u32x2_bits b = __builtin_bit_cast(lowp::u32x2_bits, q);
    return u32x4{a[0], a[1], b[0], b[1]};
  };
  row[g / 4 * 8 + g % 4] = join(x.hi, y.hi);
  row[g / 4 * 8 + 4 + g % 4] = join(x.lo, y.lo);
}

__global__ __launch_bounds__(kBlock) void split_paired_kernel(
    const float* __restrict__ A, int64_t M, int64_t lda, u32x4* __restrict__ pa, int64_t rows_out,
    const float* __restrict__ B, int64_t N, int64_t ldb, u32x4* __restrict__ pb, int64_t n_out,
    int64_t K, int64_t k_out, int64_t k_blocks, int64_t b_blocks) {
  const idx_t blk = block_x().index();
  const int t = (int)thread_x<kBlock>().index();
  const idx_t row_groups = k_out / 8;            // groups of a row; twice as many 16-byte groups
  if (blk < b_blocks) {
    constexpr int kR = kEncodeRows;
    const int w = t / kWave, lane = t % kWave;
    const idx_t n = blk / k_blocks * 32 + 4 * (lane % 8);
    const idx_t k = ((blk % k_blocks * 4 + w) * 8 + lane / 8) * kR;
    if (k >= k_out) return;
    f32x4 v[kR];
    load_cols<kR, false>(B, K, N, ldb, k, n, blk / k_blocks * 32 + 32 <= N, v);
    auto out = matrix(pb, n_out, 2 * row_groups);
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int h = 0; h < kR / 8; ++h) {
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = v[8 * h + j][c];
        store_pair(&out.at(n + c, 0), k / 8 + h, x);
      }
    return;
  }
  auto a = matrix(A, M, lda);
  auto out = matrix((u16x4*)pa, rows_out, 4 * row_groups);
  const idx_t per_row = k_out / 4, total = rows_out * per_row;
  const idx_t g0 = (blk - b_blocks) * (kBlock * kPairGroups) + t;
  f32x4 x[kPairGroups];
  idx_t row[kPairGroups], at[kPairGroups];
#pragma unroll
  for (int i = 0; i < kPairGroups; ++i) {
    const idx_t g = g0 + kBlock * i;
    row[i] = g / per_row;
    at[i] = g % per_row;
    const idx_t c = 4 * at[i];
    if (row[i] < M && c + 4 <= K) {
      x[i] = *(const f32x4_any*)&a.at(row[i], c);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) x[i][j] = row[i] < M && c + j < K ? a.at(row[i], c + j) : 0.f;
    }
  }
#pragma unroll
  for (int i = 0; i < kPairGroups; ++i) {
    if (g0 + kBlock * i >= total) continue;
    const lowp::Split4 sp = lowp::split_bf16x4(x[i][0], x[i][1], x[i][2], x[i][3]);
    const idx_t to = at[i] / 8 * 16 + at[i] % 8;       // 8 groups of hi, then 8 of lo
    out.at(row[i], to) = sp.hi;
    out.at(row[i], to + 8) = sp.lo;
  }
}

hipError_t launch_split_paired(const float* A, int64_t M, int64_t lda, void* pa, int64_t Mp,
                               const float* B, int64_t N, int64_t ldb, void* pb, int64_t Np,
                               int64_t K, int64_t Kp, hipStream_t s) {
  const int64_t k_blocks = (Kp + 511) / 512, b_blocks = k_blocks * (Np / 32);
  const int64_t a_blocks = (Mp * (Kp / 4) + kBlock * kPairGroups - 1) / (kBlock * kPairGroups);
  hipLaunchKernelGGL(split_paired_kernel, dim3((unsigned)(b_blocks + a_blocks)), dim3(kBlock),
                     0, s, A, M, lda, (u32x4*)pa, Mp, B, N, ldb, (u32x4*)pb, Np, K, Kp, k_blocks,
                     b_blocks);
  return hipGetLastError();
}

template <int kW, bool kNt>
__global__ __launch_bounds__(kBlock) void quant_cols_t_kernel(const float* __restrict__ B,
                                                              int64_t K, int64_t N, int64_t ldb,
                                                              const float* __restrict__ part,
                                                              int64_t nslices, int64_t ldp,
                                                              uint8_t* __restrict__ qt,
                                                              int64_t n_out, int64_t k_out,
                                                              int64_t ldq,
                                                              float* __restrict__ scale,
                                                              uint32_t k_blocks) {
  constexpr int kR = kEncodeRows, kWaves = kBlock / kWave;
  constexpr int kCols = 32 * (kWaves / kW), kGroups = kBlock / kCols;
  __shared__ float pmax[kGroups][kCols];
  auto thread = thread_x<kBlock>();
  const int w = (int)wave_of_block<kBlock>().index(), lane = (int)lane_of_wave().index();
  const int c4 = 32 * (w / kW) + 4 * (lane % 8);          // the thread's first column
  // k blocks of a column block follow each other; one dimension, since a second
  // one would end at 65535 of them (2^21 columns)
  const uint32_t blk = (uint32_t)block_x().index();
  const idx_t n0 = (idx_t)(blk / k_blocks) * kCols, n = n0 + c4;
  const idx_t k = ((blk % k_blocks * kW + w % kW) * 8 + lane / 8) * kR;      // and first k
  f32x4 v[kR];
  load_cols<kR, kNt>(B, K, N, ldb, k, n, n0 + kCols <= N, v);
  {
    // thread (g, c) takes slices g, g + kGroups, ... of column c
    const int c = (int)thread.index() % kCols, g = (int)thread.index() / kCols;
    auto pm = matrix(part, nslices, ldp);
    float m = 0.f;
    if (n0 + c < N)
#pragma unroll 8
      for (idx_t sl = g; sl < nslices; sl += kGroups) m = fmaxf(m, pm.at(sl, n0 + c));
    pmax[g][c] = m;
  }
  sync(thread);
  auto out = matrix(qt, n_out, ldq);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    float m = pmax[0][c4 + c];
#pragma unroll
    for (int g = 1; g < kGroups; ++g) m = fmaxf(m, pmax[g][c4 + c]);
    if (n + c >= n_out) continue;
    if (k == 0) array(scale, n_out)[n + c] = m / 448.0f;
    if (k >= k_out) continue;
    const auto e = encode_col<kR>(v, c, m > 0.f ? 448.0f / m : 1.0f, n + c < N ? K - k : 0);
    if (k + kR <= k_out) {
      *(u32x4_any*)&out.at(n + c, k) = e;
    } else {
#pragma unroll
      for (int j = 0; j < kR; ++j)
        if (k + j < k_out) out.at(n + c, k + j) = (uint8_t)(e[j / 4] >> (8 * (j % 4)));
    }
  }
}

// Which encode: the LDS tiles up to 8192 of them, since they make four times
// the blocks (3072 x 512 6.1 us against 7.9, 2560 x 3072 12.3 / 15.7, 4096 x
// 4096 18.5 both); up to 2048 where their loads are single ones, B starting off a
// 16-byte boundary.  Rows that each start at another offset from one cost the
// 16-byte loads more than single ones (an FP8 product of 300 rows with 6295
// columns at K = 4916 149 us in LDS tiles, 160 without; 12001 at K = 4099 220 and
// 263), up to about K = 6000 (5001 columns at K = 8000 187 and 174).
template <bool kNt>
hipError_t launch_cols_t(const float* B, int64_t K, int64_t N, int64_t ldb, const float* part,
                         int64_t nslices, int64_t ldp, uint8_t* qt, int64_t n_out, int64_t k_out,
                         int64_t ldq, float* scale, bool vec_in, bool vec_out, hipStream_t s) {
  const int64_t tk = (k_out + 63) / 64, tn = (n_out + 63) / 64;
  const bool odd_rows = ldb % 4 != 0 && k_out <= 6144 && tn <= 65535;
  if (tk * tn <= 2048 || (tk * tn <= 8192 && vec_in) || odd_rows) {
    hipLaunchKernelGGL(quant_cols_tile_kernel, dim3((unsigned)tk, (unsigned)tn), dim3(kBlock), 0, s,
                       B, K, N, ldb, part, nslices, ldp, qt, n_out, k_out, ldq, scale, vec_in,
                       vec_out);
    return hipGetLastError();
  }
  const bool wide = k_out >= 512;         // blocks of 512 k x 32 columns, or 128 x 128
  const int64_t kb = wide ? (k_out + 511) / 512 : (k_out + 127) / 128;
  const int64_t blocks = kb * (wide ? (n_out + 31) / 32 : (n_out + 127) / 128);
  if (!launch::grid_fits(blocks, kBlock)) return hipErrorInvalidConfiguration;
  if (wide)
    hipLaunchKernelGGL((quant_cols_t_kernel<4, kNt>), dim3((unsigned)blocks), dim3(kBlock), 0, s, B,
                       K, N, ldb, part, nslices, ldp, qt, n_out, k_out, ldq, scale, (uint32_t)kb);
  else
    hipLaunchKernelGGL((quant_cols_t_kernel<1, kNt>), dim3((unsigned)blocks), dim3(kBlock), 0, s, B,
                       K, N, ldb, part, nslices, ldp, qt, n_out, k_out, ldq, scale, (uint32_t)kb);
  return hipGetLastError();
}

int64_t colmax_slices(int64_t K, int64_t N) {
  const int64_t cblocks = (N + 4 * kBlock - 1) / (4 * kBlock);
  int64_t s = 256 / (cblocks > 0 ? cblocks : 1);
  const int64_t kmax = (K + 63) / 64;
  if (s > kmax) s = kmax;
  return s < 1 ? 1 : s;
}

// ------------------------------------------------------------------ e4m3, one pass
// The FP8 GEMM's whole pre-pass in one launch, for K up to 2048: a block holds
// a strip of 16 columns of B in registers, so B is read once, for the maxima
// and the codes (the two launches above read it twice), beside blocks of eight
// rows of A, one per wave.  512 threads; a thread of a strip holds kR
// consecutive k of four columns and stores kR codes of a column at once.  16
// columns make 64-byte row segments: the other half of a line is the
// neighbouring strip's, which runs on the same XCD (strips of an XCD are
// consecutive; 22 us against 26 at 4096 x 4096 x 2048 without).  Against the
// two launches: 4096 x 4096 x 512 9 / 17 us, 1024 10.6 / 19, 2048 22 / 25; the
// strips of K = 4096 (128 value registers, one block a CU) took 43 against 45,
// and with the encode in whole lines above the two launches are ahead there.
constexpr int kOnceBlock = 512, kOnceWaves = kOnceBlock / kWave, kStripCols = 16;

template <int kR>
struct OnceCfg {
  static constexpr int r = kR;
  static constexpr int max_k = kOnceWaves * 16 * kR;
  static constexpr int row_vecs = max_k / (4 * kWave);   // float4 per lane of a row of A
  struct Shared {
    float wave_max[kOnceWaves][kStripCols];
  };
};

template <class C>
__device__ __forceinline__ void quant_strip(const float* __restrict__ B, int64_t K, int64_t N,
                                            int64_t ldb, uint8_t* __restrict__ qt, int64_t n_out,
                                            int64_t k_out, float* __restrict__ scale, idx_t strip,
                                            typename C::Shared& sh) {
  auto thread = thread_x<kOnceBlock>();
  const int w = (int)wave_of_block<kOnceBlock>().index();
  const int lane = (int)lane_of_wave().index();
  const int c4 = 4 * (lane % 4);                          // the thread's first column of the strip
  const idx_t k = (w * 16 + lane / 4) * C::r;             // and its first k
  const idx_t n0 = strip * kStripCols;
  f32x4 v[C::r];
  load_cols<C::r, false>(B, K, N, ldb, k, n0 + c4, n0 + kStripCols <= N, v);
  f32x4 m = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < C::r; ++j)
#pragma unroll
    for (int c = 0; c < 4; ++c) m[c] = fmaxf(m[c], fabsf(v[j][c]));
#pragma unroll
  for (int c = 0; c < 4; ++c) {
#pragma unroll
    for (int s = 32; s >= 4; s >>= 1) m[c] = fmaxf(m[c], __shfl_xor(m[c], s, kWave));
    if (lane < 4) sh.wave_max[w][c4 + c] = m[c];
  }
  sync(thread);
  auto out = matrix(qt, n_out, k_out);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    float x = sh.wave_max[0][c4 + c];
#pragma unroll
    for (int i = 1; i < kOnceWaves; ++i) x = fmaxf(x, sh.wave_max[i][c4 + c]);
    if (k == 0) array(scale, n_out)[n0 + c4 + c] = x / 448.0f;
    if (k < k_out) {
      const auto e =
          encode_col<C::r>(v, c, x > 0.f ? 448.0f / x : 1.0f, n0 + c4 + c < N ? K - k : 0);
      *(std::remove_const_t<decltype(e)>*)&out.at(n0 + c4 + c, k) = e;
    }
  }
}

// Row r of A by one wave.
template <class C>
__device__ __forceinline__ void quant_row_wave(const float* __restrict__ A, int64_t M, int64_t K,
                                               int64_t lda, uint8_t* __restrict__ q,
                                               int64_t rows_out, int64_t k_out,
                                               float* __restrict__ scale, idx_t r) {
  const int lane = (int)lane_of_wave().index();
  auto a = matrix(A, M, lda);
  auto qr = matrix(q, rows_out, k_out).idx(r);
  f32x4 v[C::row_vecs];
  float amax = 0.f;
#pragma unroll
  for (int i = 0; i < C::row_vecs; ++i) {
    const idx_t c = 4 * (lane + kWave * i);
    if (r < M && 4 * kWave * (i + 1) <= K) {
      v[i] = *(const f32x4_any*)&a.at(r, c);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[i][j] = r < M && c + j < K ? a.at(r, c + j) : 0.f;
    }
  }
#pragma unroll
  for (int i = 0; i < C::row_vecs; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) amax = fmaxf(amax, fabsf(v[i][j]));
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) amax = fmaxf(amax, __shfl_xor(amax, s, kWave));
  const float inv = amax > 0.f ? 448.0f / amax : 1.0f;
#pragma unroll
  for (int i = 0; i < C::row_vecs; ++i) {
    const idx_t c = 4 * (lane + kWave * i);
    if (c >= k_out) continue;
    const uint32_t e = lowp::e4m3x4(v[i][0] * inv, v[i][1] * inv, v[i][2] * inv, v[i][3] * inv);
    *(uint32_t*)&qr[c] = e & code_mask(r < M ? K - c : 0);
  }
  if (lane == 0) array(scale, rows_out)[r] = amax / 448.0f;
}

template <class C>
__global__ __launch_bounds__(kOnceBlock) void fp8_once_kernel(
    const float* __restrict__ A, int64_t M, int64_t lda, uint8_t* __restrict__ qa,
    int64_t rows_out, float* __restrict__ sa, const float* __restrict__ B, int64_t N, int64_t ldb,
    uint8_t* __restrict__ qb, int64_t n_out, float* __restrict__ sb, int64_t K, int64_t k_out) {
  __shared__ typename C::Shared sh;
  const idx_t blk = block_x().index(), strips = n_out / kStripCols;
  if (blk < strips)
    quant_strip<C>(B, K, N, ldb, qb, n_out, k_out, sb, blk % 8 * (strips / 8) + blk / 8, sh);
  else
    quant_row_wave<C>(A, M, K, lda, qa, rows_out, k_out, sa,
                      (blk - strips) * kOnceWaves + wave_of_block<kOnceBlock>().index());
}

template <class C>
hipError_t launch_fp8_once(const float* A, int64_t M, int64_t lda, uint8_t* qa, int64_t Mp,
                           float* sa, const float* B, int64_t N, int64_t ldb, uint8_t* qb,
                           int64_t Np, float* sb, int64_t K, int64_t Kp, hipStream_t s) {
  const int64_t blocks = Np / kStripCols + Mp / kOnceWaves;
  if (!launch::grid_fits(blocks, kOnceBlock)) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL(fp8_once_kernel<C>, dim3((unsigned)blocks), dim3(kOnceBlock), 0, s, A, M, lda,
                     qa, Mp, sa, B, N, ldb, qb, Np, sb, K, Kp);
  return hipGetLastError();
}

// ------------------------------------------------------------------ GEMM launch
template <class C, bool kBuf>
__global__ __launch_bounds__(C::threads) void gemm_nt_kernel(NtOperands p, int64_t tiles_m,
                                                             int64_t tiles_n) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[C::lds_bytes];
  const idx_t t = gemm_f32::xcd_tile(block_x(), tiles_m, tiles_n);
  gemm_nt::tile<C, kBuf>(p, t / tiles_n, t % tiles_n, lds);
}

// Split-BF16 tiles straight from the FP32 operands (no pre-pass).
template <class C, bool kVec>
__global__ __launch_bounds__(C::threads) void gemm_split_kernel(gemm_nt::F32Operands f,
                                                                float* __restrict__ Cm,
                                                                int64_t ldc, int64_t tiles_m,
                                                                int64_t tiles_n) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[C::lds_bytes];
  const idx_t t = gemm_f32::xcd_tile(block_x(), tiles_m, tiles_n);
  gemm_nt::tile_split<C, kVec>(f, Cm, ldc, t / tiles_n, t % tiles_n, lds);
}

template <class C>
hipError_t launch_split(const gemm_nt::F32Operands& f, float* Cm, int64_t ldc, hipStream_t s) {
  const int64_t tm = (f.M + C::bm - 1) / C::bm, tn = (f.N + C::bn - 1) / C::bn;
  if (gemm_f32::vec_ok(f.A, f.lda, f.A, f.lda) && f.K % 4 == 0)
    hipLaunchKernelGGL((gemm_split_kernel<C, true>), dim3((unsigned)(tm * tn)), dim3(C::threads),
                       0, s, f, Cm, ldc, tm, tn);
  else
    hipLaunchKernelGGL((gemm_split_kernel<C, false>), dim3((unsigned)(tm * tn)),
                       dim3(C::threads), 0, s, f, Cm, ldc, tm, tn);
  return hipGetLastError();
}

// The buffer-range loads need a tile's rows of a plane to span less than
// 2^31 bytes (K up to about 8M FP8 or 4M BF16 values at 256-row tiles).
template <class C>
hipError_t launch_nt(const NtOperands& p, int64_t Mp, int64_t Np, hipStream_t s) {
  const int64_t tm = Mp / C::bm, tn = Np / C::bn;
  const int64_t rows = C::bm > C::bn ? C::bm : C::bn;
  if (rows * p.row_bytes < (int64_t(1) << 31))
    hipLaunchKernelGGL((gemm_nt_kernel<C, true>), dim3((unsigned)(tm * tn)), dim3(C::threads), 0,
                       s, p, tm, tn);
  else
    hipLaunchKernelGGL((gemm_nt_kernel<C, false>), dim3((unsigned)(tm * tn)), dim3(C::threads), 0,
                       s, p, tm, tn);
  return hipGetLastError();
}

// 256 x 256 tiles staged to LDS directly (gemm_dma.hpp).
template <class C, bool kNt>
__global__ __launch_bounds__(C::threads) void gemm_dma_kernel(NtOperands p, int64_t tiles_m,
                                                              int64_t tiles_n) {
  // two arrays: the compiler then sees that one stage's loads do not write
  // what the other's reads read, and waits only at the barrier
  __shared__ u32x4 even[C::stage_chunks], odd[C::stage_chunks];
  const idx_t t = gemm_f32::xcd_tile(block_x(), tiles_m, tiles_n);
  gemm_nt::dma_tile<C, kNt>(p, t / tiles_n, t % tiles_n, even, odd);
}

// `bytes`: the call's operands, planes and result.  Beyond the 256 MB that the
// memory-side cache holds, C goes past it (non-temporal stores), which leaves
// it to the planes: split BF16 4096^3 (335 MB) 2 to 5 % faster, FP8 8192^3 2 %;
// below, C is better kept: FP8 4096^3 (235 MB) 107 us against 104.
template <class Mode>
hipError_t launch_dma(const NtOperands& p, int64_t Mp, int64_t Np, int64_t bytes, hipStream_t s) {
  using C = DmaCfg<Mode>;
  const int64_t tm = Mp / C::bm, tn = Np / C::bn;
  if (bytes > (int64_t(256) << 20))
    hipLaunchKernelGGL((gemm_dma_kernel<C, true>), dim3((unsigned)(tm * tn)), dim3(C::threads), 0, s,
                       p, tm, tn);
  else
    hipLaunchKernelGGL((gemm_dma_kernel<C, false>), dim3((unsigned)(tm * tn)), dim3(C::threads), 0,
                       s, p, tm, tn);
  return hipGetLastError();
}
// A tile's rows span less than 2^31 bytes of a plane and less than 2^30 of C.
bool dma_fits(int64_t row_bytes, int64_t ldc) {
  return row_bytes < (int64_t(1) << 23) && ldc < (int64_t(1) << 20);
}

// One launch from the FP32 operands (gemm_fp8_fused.hpp).
__global__ __launch_bounds__(64 * gemm_fp8::kFusedWaves) void gemm_fp8_fused_kernel(
    const float* __restrict__ A, int64_t lda, const float* __restrict__ B, int64_t ldb,
    float* __restrict__ Cm, int64_t ldc, int64_t M, int64_t N, int64_t K) {
  __shared__ gemm_fp8::FusedLds lds;
  constexpr int T = gemm_fp8::kFusedTile;
  const auto t = layout::xcd_run_tile(block_x().index(), (M + T - 1) / T, (N + T - 1) / T);
  gemm_fp8::fused_tile(GemmProblemF32{A, lda, B, ldb, Cm, ldc, M, N, K}, t.m, t.n, lds);
}

hipError_t launch_fp8_fused(const GemmProblemF32& g, hipStream_t s) {
  constexpr int T = gemm_fp8::kFusedTile;
  const int64_t tiles = ((g.M + T - 1) / T) * ((g.N + T - 1) / T);
  hipLaunchKernelGGL(gemm_fp8_fused_kernel, dim3((unsigned)tiles),
                     dim3(64 * gemm_fp8::kFusedWaves), 0, s, g.A, g.lda, g.B, g.ldb, g.C, g.ldc,
                     g.M, g.N, g.K);
  return hipGetLastError();
}

// The direct tile over the planes (gemm_direct_nt.hpp).
template <class C>
__global__ __launch_bounds__(C::threads) void gemm_direct_nt_kernel(NtOperands p) {
  __shared__ float lds[C::lds_floats];
  const auto t = layout::xcd_run_tile(block_x().index(), (p.M + C::bm - 1) / C::bm,
                                      (p.N + C::bn - 1) / C::bn);
  gemm_nt::direct_tile<C>(p, t.m, t.n, lds);
}

template <class C>
hipError_t launch_direct_nt(const NtOperands& p, hipStream_t s) {
  const int64_t tiles = ((p.M + C::bm - 1) / C::bm) * ((p.N + C::bn - 1) / C::bn);
  hipLaunchKernelGGL(gemm_direct_nt_kernel<C>, dim3((unsigned)tiles), dim3(C::threads), 0, s, p);
  return hipGetLastError();
}

struct LowpLayout {
  int64_t Mp, Np, Kp;
  size_t a_plane, b_plane;       // bytes of one operand plane
  size_t off[8];                 // byte offsets of the workspace parts
  size_t total;
};

// bf16x3: Ah, Al, Bh^T, Bl^T.  fp8: qA, qB^T, sA, sB, column partials.
LowpLayout lowp_layout(int mode, int64_t M, int64_t N, int64_t K) {
  LowpLayout L{};
  L.Mp = round_up(M > 0 ? M : 1, kPadMN);
  L.Np = round_up(N > 0 ? N : 1, kPadMN);
  L.Kp = round_up(K > 0 ? K : 1, kPadK);
  const size_t es = mode == 1 ? 2 : 1;
  L.a_plane = align256((size_t)L.Mp * L.Kp * es);
  L.b_plane = align256((size_t)L.Np * L.Kp * es);
  size_t o = 0;
  if (mode == 1) {
    L.off[0] = o; o += L.a_plane;
    L.off[1] = o; o += L.a_plane;
    L.off[2] = o; o += L.b_plane;
    L.off[3] = o; o += L.b_plane;
  } else {
    L.off[0] = o; o += L.a_plane;
    L.off[2] = o; o += L.b_plane;
    L.off[4] = o; o += align256((size_t)L.Mp * 4);
    L.off[5] = o; o += align256((size_t)L.Np * 4);
    L.off[6] = o; o += align256((size_t)colmax_slices(K, N) * L.Np * 4);
  }
  L.total = o;
  return L;
}

unsigned grid_for(int64_t items) {
  int64_t g = (items + kBlock - 1) / kBlock;
  if (g > 8192) g = 8192;
  return (unsigned)(g < 1 ? 1 : g);
}

// The split-BF16 direct forms (direct_forms.hpp).
constexpr DirectForm kDirect[] = {
    direct<true, 4, 4, 2, 2, 1, 1>(41.8),   // 128 x 128
    direct<true, 4, 4, 1, 2, 2, 1>(20.1),   // 64 x 128
    direct<true, 4, 4, 2, 1, 2, 1>(20.4),   // 128 x 64
    direct<true, 4, 4, 1, 1, 4, 1>(10.7),   // 64 x 64
    direct<true, 3, 3, 1, 1, 4, 2>(9.3),    // 48 x 48
    direct<true, 2, 4, 1, 1, 4, 2>(7.2),    // 32 x 64
    direct<true, 2, 2, 1, 1, 4, 3>(6.3),    // 32 x 32
    direct<true, 1, 4, 1, 1, 4, 2>(4.3),    // 16 x 64
    direct<true, 1, 2, 1, 1, 8, 3>(3.9),    // 16 x 32
    direct<true, 2, 1, 1, 1, 8, 3>(4.5),    // 32 x 16
    direct<true, 1, 1, 1, 1, 16, 2>(2.3),   // 16 x 16
};
constexpr int kDirectForms = (int)(sizeof(kDirect) / sizeof(kDirect[0]));

// Times of the fused forms by the tiles a CU gets (us, K in the formulas per
// 1000).  128 x 128, two blocks a CU: 35 K for one tile, 50 K for two, 84 K
// for three, 104 K for four, 117 K for five, and 3 us of ends a tile (1000 x 1500 x 777 36 us
// against 22.5 in 64 x 128 direct tiles; 2048^3 80 against 92).  256 x 256,
// eight waves: 68 K a round, 88 K when every CU has one, and 11 us of ends
// (4096^3 366 us against 430 in 128 x 128 tiles, 3001 x 2777 x 2501 201
// against 214, 2560 x 2560 x 1024 85 against 54).
double fused128_us(int64_t M, int64_t N, int64_t K) {
  const double tiles = (double)((M + 127) / 128) * (double)((N + 127) / 128);
  const double each = tiles <= 256 ? 1.0 : (double)(int64_t)((tiles + 255) / 256);
  const double pairs = (double)(int64_t)(each / 2), odd = each - 2 * pairs;
  return (pairs * 50.0 + odd * (pairs < 2 ? 35.0 : 17.0)) * K * 1e-3 + 3.0 * each;
}
double fused256_us(int64_t M, int64_t N, int64_t K) {
  const double tiles = (double)((M + 255) / 256) * (double)((N + 255) / 256);
  const double rounds = tiles <= 256 ? 1.0 : (double)(int64_t)((tiles + 255) / 256);
  return rounds * ((68.0 + 20.0 * (tiles < 256 ? tiles / 256 : 1.0)) * K * 1e-3 + 11.0);
}

// The 256 x 256 tiles staged to LDS directly (us, K per 1000), in rounds of one
// tile a CU: full rounds, and a last one of f x 256 tiles, which runs at a
// higher clock the fewer there are.
struct Rounds {
  double whole, f;
};
Rounds rounds256(int64_t M, int64_t N) {
  const double tiles = (double)((M + 255) / 256) * (double)((N + 255) / 256);
  const double whole = (double)(int64_t)(tiles / 256);
  return {whole, tiles / 256 - whole};
}
// Split BF16, with the pre-pass over the operands: 169 us at 4096 x 4096 x
// 2048 against 194 fused, 329 at 4096^3 against 366, 126 at 3072 x 3072 x 2048
// against 162, 2300 at 8192^3 against 2840; 111 at 2048^3 against 73 in 128 x
// 128 tiles, and 58 at 4096 x 4096 x 512 against 57.
double split_dma_us(int64_t M, int64_t N, int64_t K) {
  const double k = K * 1e-3;
  const double pre = 7.0 + 8.0 * ((double)M * K + (double)K * N) / 7.2e6;
  const Rounds r = rounds256(M, N);
  const double full = std::max(14.0 + 64.0 * k, 24.0 + 34.0 * k);   // short K: bound by C
  return pre + r.whole * full +
         (r.f > 0 ? 11.0 + 3.0 * r.f + (40.0 + 22.0 * r.f * r.f) * k : 0.0);
}
// FP8, without the pre-pass, which its staged forms share: 4096^3 60 us
// against 75 in 128 x 128 tiles (with eight waves in 256 x 256 register-staged
// ones 75, too); 8192 x 4096 x 2048 with the pre-pass 101 against 112, 3072 x
// 3072 x 4096 77 against 86; 2048^3 43 against 33, 8192 x 4096 x 512 64
// against 58.
double fp8_dma_us(int64_t M, int64_t N, int64_t K) {
  const double k = K * 1e-3;
  const Rounds r = rounds256(M, N);
  return r.whole * (15.0 + 11.2 * k) + (r.f > 0 ? 7.0 + 10.0 * r.f + (7.3 + 3.9 * r.f) * k : 0.0);
}
double fp8_staged128_us(int64_t M, int64_t N, int64_t K) {
  const double tiles = (double)((M + 127) / 128) * (double)((N + 127) / 128);
  const double each = tiles <= 256 ? 1.0 : (double)(int64_t)((tiles + 255) / 256);
  return 5.0 + 1.8 * each + (4.2 * each - 0.5) * K * 1e-3;
}

// "_w8": eight waves (2 x 4) share the tile instead of four (2 x 2);
// "_fused": the operands split while they are staged (no pre-pass);
// "by_shape": a fused or a direct form, whichever the call's M, N and K make
// faster; "dBMxBN": that direct form (by_shape where a row of C is shorter
// than one load, or a stride is beyond the direct forms');
// "_p": fragment reads one group of matrix ops ahead (NtCfg kPipe);
// "_dma": stages loaded to LDS directly (gemm_dma.hpp).
// "by_shape" (FP8): one of the forms below by the rule of fp8_by_shape;
// "fused32x32": one launch from the FP32 operands; "d32x32", "d64x64": direct
// tiles over the planes.
constexpr const char* kNamesBf16[] = {"m128n128k32", "m256n128k32", "m128n256k32",
                                      "m256n256k32_d1", "m256n256k32_w8d1",
                                      "m128n128k32_fused", "m256n256k32_w8d1_fused",
                                      "by_shape", "d128x128", "d64x128", "d128x64", "d64x64",
                                      "d48x48", "d32x64", "d32x32", "d16x64", "d16x32", "d32x16",
                                      "d16x16", "m256n256k32_dma"};
constexpr int kByShape = 7, kCountBf16 = (int)(sizeof(kNamesBf16) / sizeof(kNamesBf16[0]));
constexpr int kBf16Dma = kByShape + 1 + kDirectForms;
static_assert(kCountBf16 == kBf16Dma + 1, "one name per configuration");
constexpr int kDefaultsBf16[tune::kClasses] = {kByShape, kByShape, kByShape, kByShape};
constexpr const char* kNamesFp8[] = {"m128n128k128", "m128n128k64", "m256n128k128",
                                     "m128n256k128", "m256n128k64", "m256n256k64_w8d1",
                                     "m256n256k128_w8d1", "m256n256k128_w8d1_p", "m128n128k128_p",
                                     "by_shape", "fused32x32", "d32x32", "d64x64",
                                     "m256n256k128_dma"};
constexpr int kFp8ByShape = 9, kCountFp8 = (int)(sizeof(kNamesFp8) / sizeof(kNamesFp8[0]));
constexpr int kDefaultsFp8[tune::kClasses] = {kFp8ByShape, kFp8ByShape, kFp8ByShape, kFp8ByShape};
constexpr int kFp8Fused = 10, kFp8D64 = 12, kFp8Dma = 13;
using Fp8D32 = DirectNtCfg<1, 1, 16, 2>;
using Fp8D64 = DirectNtCfg<2, 2, 8, 1>;

// The FP8 form of a call.  With up to 256 tiles of 32 x 32 (one a CU) and K in
// the registers of one block, the one-launch form saves two launches (64^3 8.2
// us against 10.3 in the staged tiles, 16 x 8000 x 512 8.2 / 13.2); up to 512 tiles
// only where one operand has a single tile of rows, so that the other is read
// once, and K is long enough to pay for its words (16 x 16000: K = 256 13.2 / 12.0
// in 64 x 64 direct tiles, 512 14.4 / 15.9, 1024 20.9 / 24.3; but 128 x 4096 x 64 16.3 /
// 9.7, 700 x 700 x 300 16.5 / 10.5, where every tile reads both operands again).
// With up to 256 tiles of 32 x 32, then of 64 x 64,
// the direct tiles share K among 16 or 8 waves (64 x 64 x 4096 22 against 36
// us, 128 x 2048 x 2048 20.5 against 27, 1024 x 1024 x 4096 34 against 37).
// Beyond that the LDS-staged tiles: 128 x 128 or the direct-to-LDS 256 x 256
// by the times above, for small M N K 128 x 128 with shorter stages.
int fp8_by_shape(int64_t M, int64_t N, int64_t K, int cls) {
  auto tiles = [&](int64_t t) { return (double)((M + t - 1) / t) * (double)((N + t - 1) / t); };
  constexpr int64_t kOnce = gemm_fp8::kFusedWaves * gemm_fp8::kFusedStep;
  if (tiles(32) <= 256 && K <= kOnce) return kFp8Fused;
  if (tiles(32) <= 512 && std::min(M, N) <= 32 && K > kOnce / 4 && K <= kOnce) return kFp8Fused;
  if (tiles(32) <= 256) return kFp8Fused + 1;
  if (tiles(64) <= 256) return kFp8D64;
  if (cls < 2) return cls == 0 ? 1 : 0;
  return fp8_dma_us(M, N, K) < fp8_staged128_us(M, N, K) ? kFp8Dma : 8;
}

const bool kRegistered =
    (tune::register_op(tune::kGemmBf16x3, "gemm_bf16x3", kCountBf16, kNamesBf16, kDefaultsBf16),
     tune::register_op(tune::kGemmFp8, "gemm_fp8", kCountFp8, kNamesFp8, kDefaultsFp8), true);

}  // namespace

namespace launch {

size_t gemm_lowp_workspace(int mode, int64_t M, int64_t N, int64_t K) {
  return lowp_layout(mode, M, N, K).total;
}

bool f4_ok(const void* p, int64_t ld) { return ((uintptr_t)p % 16) == 0 && ld % 4 == 0; }
bool w_ok(const void* p, int64_t ld, int64_t es) {   // 4 elements of es bytes per store
  return ((uintptr_t)p % (4 * es)) == 0 && ld % 4 == 0;
}

hipError_t split_bf16_rows(const float* A, int64_t M, int64_t K, int64_t lda, uint16_t* hi,
                           uint16_t* lo, int64_t ldh, hipStream_t s) {
  hipLaunchKernelGGL(split_rows_kernel, dim3(grid_for(M * ((K + 3) / 4))), dim3(kBlock), 0, s, A,
                     M, K, lda, hi, lo, M, K, ldh, f4_ok(A, lda),
                     w_ok(hi, ldh, 2) && w_ok(lo, ldh, 2));
  return hipGetLastError();
}

hipError_t split_bf16_cols(const float* B, int64_t K, int64_t N, int64_t ldb, uint16_t* hi_t,
                           uint16_t* lo_t, int64_t ldh, hipStream_t s) {
  const dim3 grid((unsigned)((K + 63) / 64), (unsigned)((N + 63) / 64));
  hipLaunchKernelGGL(split_cols_t_kernel, grid, dim3(kBlock), 0, s, B, K, N, ldb, hi_t, lo_t, N,
                     K, ldh, f4_ok(B, ldb), w_ok(hi_t, ldh, 2) && w_ok(lo_t, ldh, 2));
  return hipGetLastError();
}

hipError_t quant_e4m3_rows(const float* A, int64_t M, int64_t K, int64_t lda, uint8_t* q,
                           int64_t ldq, float* scale, hipStream_t s) {
  // a block a row, at most as many rows a launch as one grid counts
  constexpr int64_t kRows = int64_t(1) << 23;
  const bool vec_in = f4_ok(A, lda), vec_out = w_ok(q, ldq, 1);
  for (int64_t r = 0; r < M; r += kRows) {
    const int64_t rows = M - r < kRows ? M - r : kRows;
    hipLaunchKernelGGL(quant_rows_kernel, dim3((unsigned)rows), dim3(kBlock), 0, s, A + r * lda,
                       rows, K, lda, q + r * ldq, K, ldq, scale + r, vec_in, vec_out);
  }
  return hipGetLastError();
}

size_t quant_e4m3_cols_workspace(int64_t K, int64_t N) {
  return (size_t)colmax_slices(K, N) * (size_t)(N > 0 ? N : 1) * 4;
}

hipError_t quant_e4m3_cols(const float* B, int64_t K, int64_t N, int64_t ldb, uint8_t* qt,
                           int64_t ldq, float* scale, void* ws, hipStream_t s) {
  const int64_t S = colmax_slices(K, N), rows_per = (K + S - 1) / S;
  float* part = (float*)ws;
  hipLaunchKernelGGL(colmax_partial_kernel,
                     dim3((unsigned)((N + 4 * kBlock - 1) / (4 * kBlock)), (unsigned)S),
                     dim3(kBlock), 0, s, B, K, N, ldb, rows_per, part, N, f4_ok(B, ldb));
  return launch_cols_t<false>(B, K, N, ldb, part, S, N, qt, N, K, ldq, scale, f4_ok(B, ldb),
                              w_ok(qt, ldq, 1), s);
}

hipError_t gemm_bf16x3(const float* A, int64_t lda, const float* B, int64_t ldb, float* Cm,
                       int64_t ldc, int64_t M, int64_t N, int64_t K, void* ws, hipStream_t s) {
  (void)kRegistered;
  int cfg = tune::get(tune::kGemmBf16x3, tune::size_class(tune::kGemmBf16x3, M * N * K));
  const LowpLayout L = lowp_layout(1, M, N, K);
  const bool dma_ok = dma_fits(L.Kp * 4, ldc);
  if (cfg == kBf16Dma && !dma_ok) cfg = kByShape;
  if (cfg >= kByShape && cfg < kBf16Dma) {
    const double fused = std::min(fused128_us(M, N, K), fused256_us(M, N, K));
    const double dma = dma_ok && K > 0 ? split_dma_us(M, N, K) : INFINITY;
    if (K > 0 && lda <= kDirectMaxLd && ldb <= kDirectMaxLd) {
      const GemmProblemF32 g{A, lda, B, ldb, Cm, ldc, M, N, K};
      if (cfg > kByShape && kDirect[cfg - kByShape - 1].takes(M, N))
        return kDirect[cfg - kByShape - 1].launch(g, s);
      double us = 0;
      const DirectForm* d = best_direct(kDirect, kDirectForms, M, N, K, false, &us);
      // below one stage of K (32) the direct form reads word by word, the fused
      // one in 16-byte groups where A's rows are whole ones: 768000 x 32 x 16 57 us
      // against 70, 3200 x 512 x 24 5.8 / 7.1 (of K = 12 even, 25600 x 64 6.9 / 6.4)
      if (K >= 16 && K < 32 && K % 4 == 0 && gemm_f32::vec_ok(A, lda, A, lda)) us = 1.25 * us + 0.3;
      if (d && us <= fused && us <= dma) return d->launch(g, s);
    }
    cfg = dma < fused ? kBf16Dma : fused256_us(M, N, K) < fused128_us(M, N, K) ? 6 : 5;
  }
  if (cfg >= 5 && cfg < kBf16Dma && K > 0 && lda <= gemm_nt::kSplitMaxLd && ldb <= gemm_nt::kSplitMaxLd) {
    const gemm_nt::F32Operands f{A, lda, B, ldb, M, N, K};
    if (cfg == 6) return launch_split<NtCfg<256, 256, 64, Bf16x3Mode, 1, 2, 4>>(f, Cm, ldc, s);
    return launch_split<NtCfg<128, 128, 64, Bf16x3Mode>>(f, Cm, ldc, s);
  }
  // the pre-pass forms (also the fused configurations' path for K = 0 and
  // strides past the split source's limit)
  uint8_t* w = (uint8_t*)ws;
  uint16_t *ah = (uint16_t*)(w + L.off[0]), *al = (uint16_t*)(w + L.off[1]);
  uint16_t *bh = (uint16_t*)(w + L.off[2]), *bl = (uint16_t*)(w + L.off[3]);
  if (cfg == kBf16Dma) {
    const int64_t bytes = 4 * (M * K + K * N + M * N) + (int64_t)L.total;
    const hipError_t e =
        launch_split_paired(A, M, lda, ah, L.Mp, B, N, ldb, bh, L.Np, K, L.Kp, s);
    if (e != hipSuccess) return e;
    return launch_dma<Bf16x3Mode>(NtOperands{{(const uint8_t*)ah, nullptr},
                                             {(const uint8_t*)bh, nullptr},
                                             L.Kp * 4, Cm, ldc, M, N, nullptr, nullptr},
                                  L.Mp, L.Np, bytes, s);
  }
  hipLaunchKernelGGL(split_rows_kernel, dim3(grid_for(L.Mp * (L.Kp / 4))), dim3(kBlock), 0, s, A,
                     M, K, lda, ah, al, L.Mp, L.Kp, L.Kp, f4_ok(A, lda), true);
  hipLaunchKernelGGL(split_cols_t_kernel, dim3((unsigned)(L.Kp / 64), (unsigned)(L.Np / 64)),
                     dim3(kBlock), 0, s, B, K, N, ldb, bh, bl, L.Np, L.Kp, L.Kp, f4_ok(B, ldb), true);
  NtOperands p{{(const uint8_t*)ah, (const uint8_t*)al},
               {(const uint8_t*)bh, (const uint8_t*)bl},
               L.Kp * 2, Cm, ldc, M, N, nullptr, nullptr};
  switch (cfg) {
    case 1: return launch_nt<NtCfg<256, 128, 64, Bf16x3Mode>>(p, L.Mp, L.Np, s);
    case 2: return launch_nt<NtCfg<128, 256, 64, Bf16x3Mode>>(p, L.Mp, L.Np, s);
    case 3: return launch_nt<NtCfg<256, 256, 64, Bf16x3Mode, 1>>(p, L.Mp, L.Np, s);
    case 4:
    case 6: return launch_nt<NtCfg<256, 256, 64, Bf16x3Mode, 1, 2, 4>>(p, L.Mp, L.Np, s);
    default: return launch_nt<NtCfg<128, 128, 64, Bf16x3Mode>>(p, L.Mp, L.Np, s);
  }
}

hipError_t gemm_fp8(const float* A, int64_t lda, const float* B, int64_t ldb, float* Cm,
                    int64_t ldc, int64_t M, int64_t N, int64_t K, void* ws, hipStream_t s) {
  (void)kRegistered;
  const int cls = tune::size_class(tune::kGemmFp8, M * N * K);
  int cfg = tune::get(tune::kGemmFp8, cls);
  if (cfg == kFp8ByShape) cfg = fp8_by_shape(M, N, K, cls);
  if (cfg == kFp8Fused && K > 0 && lda <= gemm_fp8::kFusedMaxLd && ldb <= gemm_fp8::kFusedMaxLd)
    return launch_fp8_fused(GemmProblemF32{A, lda, B, ldb, Cm, ldc, M, N, K}, s);
  const LowpLayout L = lowp_layout(2, M, N, K);
  uint8_t* w = (uint8_t*)ws;
  uint8_t *qa = w + L.off[0], *qb = w + L.off[2];
  float *sa = (float*)(w + L.off[4]), *sb = (float*)(w + L.off[5]), *part = (float*)(w + L.off[6]);
  // what the call touches; past the 256 MB of the memory-side cache A, and B
  // at its second reading, go past it (8192^3 586 against 551 us; 4096^3, 235
  // MB, 104 against 111 when its operands are there already, 111 against 105
  // when not)
  const int64_t bytes = 4 * (M * K + K * N + M * N) + (int64_t)L.total;
  auto once = [&](auto cfg_tag) {
    return launch_fp8_once<decltype(cfg_tag)>(A, M, lda, qa, L.Mp, sa, B, N, ldb, qb, L.Np, sb, K,
                                              L.Kp, s);
  };
  // One launch, unless B is wide against A and K short: a strip's block covers
  // 512 values of K, and with a quarter of it in use the two launches are ahead
  // (16 rows, K = 16: 65000 columns 23.9 us against 28.5, 400000 88 / 138, but 30000
  // 15.7 / 16.6; K = 100: 100000 columns 41.4 / 44.3, 65000 30.9 / 29.3, 100000 of 2000
  // rows 211 / 208), and of rows it makes fewer blocks (8192 x 8192 x 16 66 / 55).
  const bool wide_b = K <= 32 ? N > 40000 && N >= 16 * M : K <= 128 && N > 81920 && N >= 64 * M;
  // the product runs only over codes that were written: a pre-pass that is not
  // launched (2^26 rows; 2^24 beyond K = 2048, a block a row) ends the call
  hipError_t pre;
  if (K > 0 && L.Kp <= 2048 && !wide_b) {
    pre = L.Kp <= 512    ? once(OnceCfg<4>{})
          : L.Kp <= 1024 ? once(OnceCfg<8>{})
                         : once(OnceCfg<16>{});
  } else {
    auto two = [&](auto nt) {
      const int64_t S = colmax_slices(K, N), rows_per = (K + S - 1) / S;
      const int64_t cblocks = (L.Np + 4 * kBlock - 1) / (4 * kBlock);
      if (!launch::grid_fits(cblocks * S + L.Mp, kBlock)) return hipErrorInvalidConfiguration;
      hipLaunchKernelGGL(fp8_prepass_kernel<nt()>, dim3((unsigned)(cblocks * S + L.Mp)),
                         dim3(kBlock), 0, s, A, M, K, lda, qa, L.Mp, L.Kp, L.Kp, sa, f4_ok(A, lda),
                         B, N, ldb, rows_per, part, L.Np, f4_ok(B, ldb), cblocks, S);
      return launch_cols_t<nt()>(B, K, N, ldb, part, S, L.Np, qb, L.Np, L.Kp, L.Kp, sb,
                                 f4_ok(B, ldb), true, s);
    };
    pre = bytes > (int64_t(256) << 20) ? two(std::true_type{}) : two(std::false_type{});
  }
  if (pre != hipSuccess) return pre;
  NtOperands p{{qa, nullptr}, {qb, nullptr}, L.Kp, Cm, ldc, M, N, sa, sb};
  if (cfg == kFp8Dma) {
    if (dma_fits(p.row_bytes, ldc))
      return launch_dma<Fp8Mode>(p, L.Mp, L.Np, bytes, s);
    cfg = 7;
  }
  if (cfg >= kFp8Fused) {
    if (cfg == kFp8D64 && gemm_nt::direct_tile_ok<Fp8D64>(L.Kp))
      return launch_direct_nt<Fp8D64>(p, s);
    if (gemm_nt::direct_tile_ok<Fp8D32>(L.Kp)) return launch_direct_nt<Fp8D32>(p, s);
  }
  switch (cfg) {
    case 1: return launch_nt<NtCfg<128, 128, 64, Fp8Mode>>(p, L.Mp, L.Np, s);
    case 2: return launch_nt<NtCfg<256, 128, 128, Fp8Mode>>(p, L.Mp, L.Np, s);
    case 3: return launch_nt<NtCfg<128, 256, 128, Fp8Mode>>(p, L.Mp, L.Np, s);
    case 4: return launch_nt<NtCfg<256, 128, 64, Fp8Mode>>(p, L.Mp, L.Np, s);
    case 5: return launch_nt<NtCfg<256, 256, 64, Fp8Mode, 1, 2, 4>>(p, L.Mp, L.Np, s);
    case 6: return launch_nt<NtCfg<256, 256, 128, Fp8Mode, 1, 2, 4>>(p, L.Mp, L.Np, s);
    case 7: return launch_nt<NtCfg<256, 256, 128, Fp8Mode, 1, 2, 4, true>>(p, L.Mp, L.Np, s);
    case 8: return launch_nt<NtCfg<128, 128, 128, Fp8Mode, 2, 2, 2, true>>(p, L.Mp, L.Np, s);
    default: return launch_nt<NtCfg<128, 128, 128, Fp8Mode>>(p, L.Mp, L.Np, s);
  }
}

}  // namespace launch
}  // namespace desc
