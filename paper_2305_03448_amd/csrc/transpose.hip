// transpose.hip -- out-of-place transpose of a row-major rows x cols matrix
// of 32-bit words (the "matrix transposition" benchmark of Sec. 5 and the
// running example of Sec. 1).
//
// The structure is the paper's: every block owns one tile, its threads copy
// the tile from the input into an LDS buffer, the block synchronises, and
// the threads copy the tile back out transposed, so both the global reads
// and the global writes run along rows.  On CDNA a tile is T x T words
// (T = 32, 64 or 128; Listing 2 uses 32) and a block is 256 threads seen as
// a [256/(T/4)][T/4] block, every thread moving 16 bytes per row:
//
//   read  : thread (y, x) copies rows y, y+TY, y+2TY, ... of the tile, words
//           4x..4x+3 of each (group_by_tile::<T,T/4> over int32x4 columns,
//           then group_by_row::<T,T/TY>);
//   write : the same thread writes rows y, y+TY, ... of the transposed tile,
//           each four consecutive words being one 16-byte store, and reads
//           them from column y+TY*i, rows 4x..4x+3 of the LDS tile.
//
// The LDS tile has a row pitch of T+1 words, so that the column-wise reads
// of a wave spread over the banks.
// Blocks take the column tiles of their row of tiles in diagonal order
// (block (x, y) takes tile (x + y mod the tiles per row, y)): with the plain
// order the blocks in flight together write output rows a power-of-two
// stride apart, which measured 10-13 % slower on MI355X.
// Matrices that are not whole tiles of aligned groups take the form at the
// end of this file (transpose_any_kernel); where a side is shorter than one
// group, the tiles go through a guarded element-by-element copy with the same
// tile and barrier.
// The kernel moves bit patterns only: NaN payloads, signed zeros and
// subnormals pass unchanged.
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"
#include "layouts.hpp"
#include "tuning.hpp"
#include "view.hpp"

namespace desc {
namespace {

constexpr int kBlock = 256;

template <int kT, bool kNt, int kThreads>
struct TransposeShape {
  static constexpr int block = kThreads;     // threads per block
  static constexpr int t = kT;               // tile edge (words)
  static constexpr int pitch = kT + 1;       // LDS row pitch (words)
  static constexpr int tx = kT / 4;          // threads along a row (16 bytes each)
  static constexpr int ty = kThreads / tx;   // threads along a column
  static constexpr int items = kT / ty;      // rows per thread
  static constexpr bool nt = kNt;
  static_assert(ty * items == kT, "tile rows must divide among the thread rows");
};
// 256 threads per block, and 512 (twice the waves per tile, half the rows
// per thread).
template <int kT, bool kNt>
struct TransposeCfg : TransposeShape<kT, kNt, kBlock> {};
template <int kT, bool kNt>
struct TransposeCfg512 : TransposeShape<kT, kNt, 512> {};

template <bool kNt, class T>
__device__ __forceinline__ T load16(const T* p) {
  if constexpr (kNt) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool kNt, class T>
__device__ __forceinline__ void store16(T v, T* p) {
  if constexpr (kNt) __builtin_nontemporal_store(v, p);
  else *p = v;
}

template <class C, bool kVec>
__global__ __launch_bounds__(C::block) void transpose32_kernel(const uint32_t* __restrict__ in,
                                                             uint32_t* __restrict__ out,
                                                             int64_t rows, int64_t cols) {
  constexpr int T = C::t, TY = C::ty, TX = C::tx, IT = C::items;
  __shared__ uint32_t lds[T * C::pitch];
  // Column tile of the input in diagonal order: row tile by starts at column
  // tile by, so that the blocks in flight together write output rows spread
  // over the matrix rather than rows a power-of-two stride apart.
  const Block bx{((idx_t)blockIdx.x + (idx_t)blockIdx.y) % (idx_t)gridDim.x, (idx_t)gridDim.x};
  auto by = block_y();   // row tile of the input
  auto thread = thread_x<C::block>();
  const Block bz{(idx_t)blockIdx.z, (idx_t)gridDim.z};   // matrix of the batch

  // The LDS tile as [T][T+1] words with the padding column split off.
  auto tile = matrix(lds, T, C::pitch).template fst<1>(T);            // [T][T]

  const bool full = kVec && (by.index() + 1) * T <= rows && (bx.index() + 1) * T <= cols;
  if (full) {
    auto t2 = thread_yx<TY, TX>();
    // input tile (by, bx), as [T rows][T/4 groups of 4 words]
    auto a_mine = layout::tile_rows<T, IT>(
        matrices((const u32x4*)in, bz.count(), rows, cols / 4).select(bz), by, bx, t2.y, t2.x);
    auto l_mine = layout::lds_rows<T, IT>(tile, t2.y, t2.x);                              // [IT][4]
    u32x4 v[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) v[i] = load16<C::nt>(&a_mine[i]);
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      auto l = l_mine.idx(i);
      l[0] = v[i].x; l[1] = v[i].y; l[2] = v[i].z; l[3] = v[i].w;
    }
    sync(thread);
    // output tile (bx, by) of the cols x rows result
    auto b_mine = layout::tile_rows<T, IT>(
        matrices((u32x4*)out, bz.count(), cols, rows / 4).select(bz), bx, by, t2.y, t2.x);
    // the LDS tile read column-wise: element (i, k) = tile[4x + k][y + TY i]
    auto lt = layout::lds_cols<T, IT>(tile, t2.y, t2.x);
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      auto l = lt.idx(i);
      u32x4 w;
      w.x = l[0]; w.y = l[1]; w.z = l[2]; w.w = l[3];
      store16<C::nt>(w, &b_mine[i]);
    }
  } else {
    // Ragged edge: element e of the tile is (e / T, e % T); guard both sides.
    auto a = matrices(in, bz.count(), rows, cols).select(bz);
    auto b = matrices(out, bz.count(), cols, rows).select(bz);
    const idx_t r0 = by.index() * T, c0 = bx.index() * T;
    for (idx_t e = thread.index(); e < T * T; e += C::block) {
      const idx_t r = e / T, c = e % T;
      if (r0 + r < rows && c0 + c < cols) tile.at(r, c) = a.at(r0 + r, c0 + c);
    }
    sync(thread);
    for (idx_t e = thread.index(); e < T * T; e += C::block) {
      const idx_t c = e / T, r = e % T;
      if (r0 + r < rows && c0 + c < cols) b.at(c0 + c, r0 + r) = tile.at(r, c);
    }
  }
}

template <class E>
bool any_shape(const void* in, const void* out, int64_t rows, int64_t cols, int T);
template <class E>
hipError_t transpose_any(const void* in, void* out, int64_t batch, int64_t rows, int64_t cols,
                         hipStream_t s);
template <class E, int kT, int kThreads, bool kNt>
hipError_t launch_any(const void* in, void* out, int64_t batch, int64_t rows, int64_t cols,
                      hipStream_t s);

// kByShape: matrices that are not whole tiles take the tile that transpose_any
// picks, else C's.
template <class C, bool kByShape = false>
hipError_t launch_transpose(const uint32_t* in, uint32_t* out, int64_t batch, int64_t rows,
                            int64_t cols, hipStream_t s) {
  constexpr int T = C::t;
  if (any_shape<uint32_t>(in, out, rows, cols, T) &&
      launch::grid_fits((cols + T - 1) / T, C::block)) {
    if constexpr (kByShape) return transpose_any<uint32_t>(in, out, batch, rows, cols, s);
    else return launch_any<uint32_t, T, C::block, C::nt>(in, out, batch, rows, cols, s);
  }
  // past 2^29 columns (2^30 of a 128-wide tile of 512 threads) 128 x 128 tiles
  // of 256 threads, whose grid takes every column count the call accepts
  using Wide = TransposeCfg<128, C::nt>;
  if constexpr (!std::is_same_v<C, Wide>)
    if (!launch::grid_fits((cols + T - 1) / T, C::block))
      return launch_transpose<Wide>(in, out, batch, rows, cols, s);
  if (!launch::grid_fits((cols + T - 1) / T, C::block)) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)((cols + T - 1) / T), (unsigned)((rows + T - 1) / T),
                  (unsigned)batch);
  const bool vec = rows % 4 == 0 && cols % 4 == 0 && (((uintptr_t)in | (uintptr_t)out) & 15) == 0;
  if (vec)
    hipLaunchKernelGGL((transpose32_kernel<C, true>), grid, dim3(C::block), 0, s, in, out, rows,
                       cols);
  else
    hipLaunchKernelGGL((transpose32_kernel<C, false>), grid, dim3(C::block), 0, s, in, out, rows,
                       cols);
  return hipGetLastError();
}

// ----------------------------------------------------------------- other element sizes
// The same kernel for elements of 1, 2 or 8 bytes (the paper's own example
// moves doubles): a 16-byte group holds kV = 16 / sizeof(E) elements and a
// tile is T x T elements read by a [256 / (T/kV)][T/kV] block.  A column
// read of the LDS tile must spread over the banks: bytes pad the rows by 4
// bytes; 2- and 8-byte elements keep unpadded rows and XOR-swizzle the
// column index with the row (a whole-element pad cannot separate the 64
// rows one wave reads): doubles by c ^ ((r / 2) % 32), which gives the 32
// rows a half-wave reads 32 different 8-byte bank pairs, and 2-byte elements
// by c ^ 4 ((r / 8) % 16), which gives the 16 rows of a wave different
// dword columns while keeping element pairs in one dword.
template <class E, int kT>
struct TransposeCfgE {
  static constexpr int v = 16 / (int)sizeof(E);            // elements per 16-byte group
  static constexpr int t = kT;
  static constexpr int pad = sizeof(E) == 1 ? 4 : 0;
  static constexpr int pitch = kT + pad;
  static constexpr int tx = kT / v;
  static constexpr int ty = kBlock / tx;
  static constexpr int items = kT / ty;
  static_assert(tx * ty == kBlock && ty * items == kT, "tile rows must divide among the threads");
};

template <class C, class E, bool kVec>
__global__ __launch_bounds__(kBlock) void transpose_elem_kernel(const E* __restrict__ in,
                                                                E* __restrict__ out, int64_t rows,
                                                                int64_t cols) {
  constexpr int T = C::t, TY = C::ty, TX = C::tx, IT = C::items, V = C::v;
  typedef E vec_t __attribute__((ext_vector_type(V)));
  __shared__ __attribute__((aligned(16))) E lds[T * C::pitch];
  // Diagonal tile order: row tile by starts at column tile by, so that the
  // blocks in flight together write output rows spread over the matrix
  // rather than rows a power-of-two stride apart.
  const Block bx{((idx_t)blockIdx.x + (idx_t)blockIdx.y) % (idx_t)gridDim.x, (idx_t)gridDim.x};
  auto by = block_y();
  auto thread = thread_x<kBlock>();
  const Block bz{(idx_t)blockIdx.z, (idx_t)gridDim.z};
  auto tile = [&] {
    if constexpr (sizeof(E) == 8)
      return matrix(lds, T, T).template xor_swizzle_by<2, 32, 1>();     // [T][T]
    else if constexpr (sizeof(E) == 2)
      return matrix(lds, T, T).template xor_swizzle_by<8, 16, 4>();
    else
      return matrix(lds, T, C::pitch).template fst<1>(T);
  }();

  const bool full = kVec && (by.index() + 1) * T <= rows && (bx.index() + 1) * T <= cols;
  if (full) {
    auto t2 = thread_yx<TY, TX>();
    auto a_mine = layout::tile_rows<T, IT, V>(
        matrices((const vec_t*)in, bz.count(), rows, cols / V).select(bz), by, bx, t2.y, t2.x);
    auto l_mine = layout::lds_rows<T, IT, V>(tile, t2.y, t2.x);                        // [IT][V]
    vec_t g[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) g[i] = __builtin_nontemporal_load(&a_mine[i]);
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      auto l = l_mine.idx(i);
#pragma unroll
      for (int k = 0; k < V; ++k) l[k] = g[i][k];
    }
    sync(thread);
    auto b_mine = layout::tile_rows<T, IT, V>(
        matrices((vec_t*)out, bz.count(), cols, rows / V).select(bz), bx, by, t2.y, t2.x);
    auto lt = layout::lds_cols<T, IT, V>(tile, t2.y, t2.x);
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      auto l = lt.idx(i);
      vec_t w;
#pragma unroll
      for (int k = 0; k < V; ++k) w[k] = l[k];
      __builtin_nontemporal_store(w, &b_mine[i]);
    }
  } else {
    auto a = matrices(in, bz.count(), rows, cols).select(bz);
    auto b = matrices(out, bz.count(), cols, rows).select(bz);
    const idx_t r0 = by.index() * T, c0 = bx.index() * T;
    for (idx_t e = thread.index(); e < T * T; e += kBlock) {
      const idx_t r = e / T, c = e % T;
      if (r0 + r < rows && c0 + c < cols) tile.at(r, c) = a.at(r0 + r, c0 + c);
    }
    sync(thread);
    for (idx_t e = thread.index(); e < T * T; e += kBlock) {
      const idx_t c = e / T, r = e % T;
      if (r0 + r < rows && c0 + c < cols) b.at(c0 + c, r0 + r) = tile.at(r, c);
    }
  }
}

// ----------------------------------------------------------------- any shape
// The form for matrices that are not whole tiles of 16-byte groups: odd row
// lengths, unaligned matrices, ragged edges.  The same tiles, threads and
// swizzles, with 16-byte accesses at element alignment (the hardware takes
// them at any address), and edges without element loops:
//   * a tile that would hold fewer than kV rows or columns starts earlier, so
//     that it holds kV of them;
//   * in a tile of hr x hc, a thread's group of kV columns (or, writing, of
//     kV rows) starts at min(kV x, hc - kV): every access is a whole group
//     inside the matrix, and two groups may move the same elements twice.
// Loads are unconditional (rows past the tile read its last row); only the
// LDS writes and the stores are guarded.
template <class E, int kT, bool kNt, int kThreads>
struct AnyShape {
  static constexpr int v = 16 / (int)sizeof(E), t = kT, block = kThreads;
  static constexpr int pad = sizeof(E) == 1 ? 4 : sizeof(E) == 4 ? 1 : 0;
  static constexpr int pitch = kT + pad;
  static constexpr int tx = kT / v, ty = kThreads / tx, items = kT / ty;
  static constexpr bool nt = kNt;
  static_assert(tx * ty == kThreads && ty * items == kT, "tile rows must divide among the threads");
};

template <class C, class E>
__global__ __launch_bounds__(C::block) void transpose_any_kernel(const E* __restrict__ in,
                                                                 E* __restrict__ out,
                                                                 int64_t rows, int64_t cols) {
  constexpr int T = C::t, TY = C::ty, TX = C::tx, IT = C::items, V = C::v;
  typedef E vec_t __attribute__((ext_vector_type(V))) __attribute__((aligned(sizeof(E))));
  __shared__ __attribute__((aligned(16))) E lds[T * C::pitch];
  const Block bx{((idx_t)blockIdx.x + (idx_t)blockIdx.y) % (idx_t)gridDim.x, (idx_t)gridDim.x};
  auto by = block_y();
  auto thread = thread_x<C::block>();
  const Block bz{(idx_t)blockIdx.z, (idx_t)gridDim.z};
  auto tile = [&] {
    if constexpr (sizeof(E) == 8)
      return matrix(lds, T, T).template xor_swizzle_by<2, 32, 1>();     // [T][T]
    else if constexpr (sizeof(E) == 2)
      return matrix(lds, T, T).template xor_swizzle_by<8, 16, 4>();
    else
      return matrix(lds, T, C::pitch).template fst<1>(T);
  }();
  auto a = matrices(in, bz.count(), rows, cols).select(bz);
  auto b = matrices(out, bz.count(), cols, rows).select(bz);
  const idx_t r0 = layout::tile_start<T, V>(by.index(), rows);
  const idx_t c0 = layout::tile_start<T, V>(bx.index(), cols);
  const int hr = (int)(rows - r0 < T ? rows - r0 : T), hc = (int)(cols - c0 < T ? cols - c0 : T);
  const int y = (int)thread.index() / TX, x = (int)thread.index() % TX;

  vec_t g[IT];
  const int gc = layout::tile_group<V>(x, hc);          // first column of the thread's group
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int r = y + TY * i;
    const vec_t* p = (const vec_t*)&a.at(r0 + (r < hr ? r : hr - 1), c0 + gc);
    if constexpr (C::nt) g[i] = __builtin_nontemporal_load(p);
    else g[i] = *p;
  }
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int r = y + TY * i;
    if (r < hr && V * x < hc) {
#pragma unroll
      for (int k = 0; k < V; ++k) tile.at(r, gc + k) = g[i][k];
    }
  }
  sync(thread);
  const int gr = layout::tile_group<V>(x, hr);          // first row of the thread's group
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int c = y + TY * i;
    if (c < hc && V * x < hr) {
      vec_t w;
#pragma unroll
      for (int k = 0; k < V; ++k) w[k] = tile.at(gr + k, c);
      vec_t* p = (vec_t*)&b.at(c0 + c, r0 + gr);
      if constexpr (C::nt) __builtin_nontemporal_store(w, p);
      else *p = w;
    }
  }
}

// Whether a call takes that form: anything but whole tiles of T x T in aligned
// groups, once both sides hold a group.  The element loops it replaces cost
// 10-15 us a launch by their latency alone: 2000 x 2000 words 17.4 -> 7.1 us,
// 100 x 200 16-bit elements 16.5 -> 3.2, a batch of 12 1000 x 777 of them
// 34.9 -> 10.4; and on unaligned matrices most of the time: 8191 x 16001
// 16-bit elements 360 -> 167 us, 8191 x 8189 words 222 -> 129 us.  Its largest
// tiles have 512 threads, so twice as many columns reach the end of a grid:
// such a matrix keeps the 256-thread form.
template <class E>
bool any_shape(const void* in, const void* out, int64_t rows, int64_t cols, int T) {
  constexpr int kV = 16 / (int)sizeof(E);
  constexpr int kLargest = sizeof(E) == 8 ? 64 : 128;
  if (!launch::grid_fits((cols + kLargest - 1) / kLargest, 512)) return false;
  const bool whole =
      rows % T == 0 && cols % T == 0 && (((uintptr_t)in | (uintptr_t)out) & 15) == 0;
  return !whole && rows >= kV && cols >= kV;
}

template <class E, int kT, int kThreads, bool kNt>
hipError_t launch_any(const void* in, void* out, int64_t batch, int64_t rows, int64_t cols,
                      hipStream_t s) {
  if (!launch::grid_fits((cols + kT - 1) / kT, kThreads)) return hipErrorInvalidConfiguration;
  using C = AnyShape<E, kT, kNt, kThreads>;
  const dim3 grid((unsigned)((cols + kT - 1) / kT), (unsigned)((rows + kT - 1) / kT),
                  (unsigned)batch);
  hipLaunchKernelGGL((transpose_any_kernel<C, E>), grid, dim3(kThreads), 0, s, (const E*)in,
                     (E*)out, rows, cols);
  return hipGetLastError();
}

// Tile by size: the largest tile writes the longest pieces of output rows and
// wins once it fills the GPU; below, smaller tiles finish sooner.  us in tiles of
// 64 and 128, for one matrix and for a batch of 12 (ragged, near-square):
//   bytes   1.1 MB 2.8 / 3.6 and 3.0 / 3.7, 4 MB 4.5 / 4.4 and 4.8 / 5.5, 8 MB 7.3 /
//           7.0 and 7.2 / 7.8, 16 MB 14.6 / 11.0 and 14.9 / 11.8
//   16 bits 1.1 MB 3.0 / 4.1 and 3.0 / 4.1, 4 MB 4.1 / 4.7 and 4.3 / 4.9, 8 MB 5.7 /
//           5.7 and 5.9 / 6.7, 16 MB 10.4 / 8.8 and 10.3 / 9.4
//   words   8 MB 4.7 / 5.4 and 4.8 / 5.9, 16 MB 7.6 / 7.3 and 7.8 / 8.6, 32 MB 13.9 /
//           12.7 and 14.1 / 13.8; 0.25 MB 2.4 in tiles of 32, 2.8 of 64
// Streaming accesses only where both arrays together outgrow the last-level
// cache (8192 x 6144 words, 403 MB: 71 us against 78; 4112^2 doubles, 271 MB: 70
// against 46) and every piece of an output row is whole 128-byte lines: two
// blocks share a line otherwise, and it must stay in the cache to be written
// once (16383 x 16381 bytes: 225 us against 197).
template <class E>
hipError_t transpose_any(const void* in, void* out, int64_t batch, int64_t rows, int64_t cols,
                         hipStream_t s) {
  const int64_t count = batch * rows * cols;
  const bool lines = rows * (int64_t)sizeof(E) % 128 == 0 && (uintptr_t)out % 128 == 0 &&
                     2 * count * (int64_t)sizeof(E) >= (int64_t)3 << 27;
  if constexpr (sizeof(E) == 8)
    return lines ? launch_any<E, 64, 512, true>(in, out, batch, rows, cols, s)
                 : launch_any<E, 64, 512, false>(in, out, batch, rows, cols, s);
  if constexpr (sizeof(E) == 4)
    if (count < (int64_t)1 << 16)
      return launch_any<E, 32, 256, false>(in, out, batch, rows, cols, s);
  if constexpr (sizeof(E) <= 4)
    if (count < (int64_t)(sizeof(E) == 4 ? 6 : 4) << 20)
      return launch_any<E, 64, 256, false>(in, out, batch, rows, cols, s);
  if constexpr (sizeof(E) <= 4)
    return lines ? launch_any<E, 128, 512, true>(in, out, batch, rows, cols, s)
                 : launch_any<E, 128, 512, false>(in, out, batch, rows, cols, s);
}

template <class E, int kT>
hipError_t launch_transpose_elem(const void* in, void* out, int64_t batch, int64_t rows,
                                 int64_t cols, hipStream_t s) {
  using C = TransposeCfgE<E, kT>;
  if (any_shape<E>(in, out, rows, cols, kT))
    return transpose_any<E>(in, out, batch, rows, cols, s);
  if (!launch::grid_fits((cols + kT - 1) / kT, kBlock)) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)((cols + kT - 1) / kT), (unsigned)((rows + kT - 1) / kT),
                  (unsigned)batch);
  const bool vec = rows % C::v == 0 && cols % C::v == 0 &&
                   (((uintptr_t)in | (uintptr_t)out) & 15) == 0;
  if (vec)
    hipLaunchKernelGGL((transpose_elem_kernel<C, E, true>), grid, dim3(kBlock), 0, s,
                       (const E*)in, (E*)out, rows, cols);
  else
    hipLaunchKernelGGL((transpose_elem_kernel<C, E, false>), grid, dim3(kBlock), 0, s,
                       (const E*)in, (E*)out, rows, cols);
  return hipGetLastError();
}

// "tT": tiles of T x T words whatever the matrix; "by_shape": the tile by size,
// of whole aligned tiles and of the others each by its own measurements.
constexpr const char* kNames[] = {"t64_nt", "t64", "t32_nt", "t32", "t128_nt", "t128",
                                   "t128_nt_b512", "t128_b512", "by_shape"};
constexpr int kByShape = 8;
constexpr int kDefaults[tune::kClasses] = {kByShape, kByShape, kByShape, kByShape};
const bool kRegistered =
    (tune::register_op(tune::kTranspose32, "transpose_32", 9, kNames, kDefaults), true);

}  // namespace

namespace launch {

// Rows are tiled by at most 128 words, so a grid of 65535 row tiles covers
// any row count this bound admits.
int64_t transpose_max_rows() { return (int64_t)65535 * 32; }

hipError_t transpose_32(const uint32_t* in, uint32_t* out, int64_t batch, int64_t rows,
                        int64_t cols, hipStream_t s) {
  if (batch == 0 || rows == 0 || cols == 0) return hipSuccess;
  (void)kRegistered;
  const int64_t size = batch * rows * cols;
  const int cls = tune::size_class(tune::kTranspose32, size);
  const int cfg = tune::get(tune::kTranspose32, cls);
  if (cfg == kByShape) {
    if (cls < 2) return launch_transpose<TransposeCfg<32, false>, true>(in, out, batch, rows, cols, s);
    if (cls < 3)
      return launch_transpose<TransposeCfg512<128, false>, true>(in, out, batch, rows, cols, s);
    return launch_transpose<TransposeCfg512<128, true>, true>(in, out, batch, rows, cols, s);
  }
  switch (cfg) {
    case 1: return launch_transpose<TransposeCfg<64, false>>(in, out, batch, rows, cols, s);
    case 2: return launch_transpose<TransposeCfg<32, true>>(in, out, batch, rows, cols, s);
    case 3: return launch_transpose<TransposeCfg<32, false>>(in, out, batch, rows, cols, s);
    case 4: return launch_transpose<TransposeCfg<128, true>>(in, out, batch, rows, cols, s);
    case 5: return launch_transpose<TransposeCfg<128, false>>(in, out, batch, rows, cols, s);
    case 6: return launch_transpose<TransposeCfg512<128, true>>(in, out, batch, rows, cols, s);
    case 7: return launch_transpose<TransposeCfg512<128, false>>(in, out, batch, rows, cols, s);
    default: return launch_transpose<TransposeCfg<64, true>>(in, out, batch, rows, cols, s);
  }
}

// Tiles of 128 elements for 1- and 2-byte elements, 64 for doubles (eight
// 16-byte groups per thread either way).
int64_t transpose_elem_max_rows(int64_t elem_bytes) {
  return (int64_t)65535 * (elem_bytes == 8 ? 64 : 128);
}

hipError_t transpose_elem(const void* in, void* out, int64_t elem_bytes, int64_t batch,
                          int64_t rows, int64_t cols, hipStream_t s) {
  if (batch == 0 || rows == 0 || cols == 0) return hipSuccess;
  switch (elem_bytes) {
    case 1: return launch_transpose_elem<uint8_t, 128>(in, out, batch, rows, cols, s);
    case 2: return launch_transpose_elem<uint16_t, 128>(in, out, batch, rows, cols, s);
    case 4:
      return transpose_32((const uint32_t*)in, (uint32_t*)out, batch, rows, cols, s);
    default: return launch_transpose_elem<uint64_t, 64>(in, out, batch, rows, cols, s);
  }
}

}  // namespace launch
}  // namespace desc
