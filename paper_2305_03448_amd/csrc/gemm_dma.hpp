// gemm_dma.hpp -- the 256 x 256 tile of the low-precision GEMMs whose stages
// go from memory to LDS without passing through registers.
//
// Four waves, one per SIMD, take 128 x 128 of the tile each: 256 accumulator
// registers, and 16 KB of LDS reads per wave and step for 16 matrix ops (FP8;
// 48 in the split-BF16 mode), where eight waves of 128 x 64 read 12 KB for
// half the ops.  A stage is 64 KB, double buffered: the loads of stage s + 2
// write LDS directly, so they take no registers and no LDS-write
// instructions, and have about a stage and a half of matrix ops to arrive.
// Fragments are read one step ahead of the matrix ops that use them.
//
// What bounds it (4096^3): FP8 1.42 us a stage, where the matrix ops alone
// take 1.10 and 1.32 without the loads, and 15 us of ends, most of it the
// 67 MB of C, which all blocks write at once; split BF16 285 to 320 us, 224 for the
// matrix ops alone: the clock falls to 1.6 GHz under them, so what the loads
// and reads cost is their energy.  The eight-wave register-staged tile takes
// 75 us (FP8), and 355 us from the FP32 operands in the split mode.  All of a
// stage's loads at the start of its second step cost 7 to 13 % more, spread
// one to a matrix op as here least.
//
// One padded plane per operand ([rows][row_bytes], zeros past K), a tile's rows
// below 2^31 bytes.  In the split mode its rows hold, for every 32 k, the 32 hi
// values and then the 32 lo values, so that a stage takes whole 128-byte lines
// of it (half lines of two planes took 160 us against 145 at 4096 x 4096 x 2048,
// and at 8192^3, with the pre-pass, 2550 against 2300).
#pragma once
#include <type_traits>

#include "gemm_nt.hpp"

namespace desc {

template <class Mode>
struct DmaCfg {
  using mode = Mode;
  static constexpr int bm = 256, bn = 256, wm = 2, wn = 2, threads = 256;
  static constexpr int wtm = bm / wm, wtn = bn / wn, fm = wtm / 32, fn = wtn / 32;
  static constexpr int steps = 2;
  static constexpr int part = steps * Mode::step_bytes;     // bytes of one value's plane (hi, lo)
  static constexpr int bkb = Mode::planes * part;           // bytes per row and stage
  static constexpr int chunks = bkb / 16;
  static constexpr int rows_per_256 = 256 / bkb;
  static constexpr int stage_chunks = (bm + bn) * chunks;   // 16-byte chunks: 64 KB
  static constexpr int rows_per_load = threads / chunks;    // rows one load of the block covers
  static constexpr int loads = bm / rows_per_load;          // per operand
  static_assert(bkb == 128, "a stage takes whole lines");
  // a load's rows start at a multiple of the swizzle's period, so a lane's
  // offset in a plane is the same for every load
  static_assert(rows_per_load % (rows_per_256 * chunks) == 0 && 32 % (rows_per_256 * chunks) == 0,
                "the swizzle repeats within a load and a fragment");
  static_assert(bm == bn && loads * rows_per_load == bm, "loads cover an operand's rows");
};

namespace gemm_nt {

// A step's fragments of one wave: 64 registers in both modes.  A fragment is
// one value, so that the registers of a matrix op's operand stay together.
template <class C>
struct StepFrags {
  using F = std::conditional_t<C::mode::lane_bytes == 32, mfma::i32x8, mfma::bf16x8>;
  F a[C::mode::planes][C::fm], b[C::mode::planes][C::fn];
};

// The block's barrier without a wait for loads: the caller has waited for
// what the barrier publishes (s_barrier orders nothing by itself, and neither
// pass of the compiler may move a memory access over it).
__device__ __forceinline__ void bare_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
}

template <int k>
using I = std::integral_constant<int, k>;

// kNt: C stored non-temporally.
template <class C, bool kNt>
__device__ __forceinline__ void dma_tile(const NtOperands& p, idx_t tm, idx_t tn, u32x4* even,
                                         u32x4* odd) {
  using Mode = typename C::mode;
  constexpr int P = Mode::planes, LB = Mode::lane_bytes, CPR = C::chunks;
  auto thread = thread_x<C::threads>();
  const int t = (int)thread.index();
  const int lane = (int)lane_of_wave().index();
  const int half = lane / 32, col32 = lane % 32;
  const int w = __builtin_amdgcn_readfirstlane((int)wave_of_block<C::threads>().index());
  const int wm = w / C::wn, wn = w % C::wn;
  const idx_t m0 = tm * C::bm, n0 = tn * C::bn;
  const idx_t nk = p.row_bytes / C::bkb;

  // LDS of a stage: [A rows then B rows][chunks], swizzled
  auto rows_of = [&](u32x4* buf) {
    return matrix(buf, C::bm + C::bn, CPR).template xor_swizzle<C::rows_per_256, CPR>();
  };

  // A load's lanes fill consecutive chunks of LDS: lane t of the block the
  // stored chunk t % CPR of row t / CPR, which holds the row's chunk
  // (t % CPR) ^ swizzle(row).
  const int row = t / CPR;
  const uint32_t lane_off = (uint32_t)row * (uint32_t)p.row_bytes +
                            16u * (uint32_t)((t % CPR) ^ ((row / C::rows_per_256) % CPR));
  const uint32_t load_off = (uint32_t)C::rows_per_load * (uint32_t)p.row_bytes;
  const uint32_t tile_bytes = (uint32_t)C::bm * (uint32_t)p.row_bytes;
  const uint8_t* first[2] = {&matrix(p.a[0], 0, p.row_bytes).at(m0, 0),
                             &matrix(p.b[0], 0, p.row_bytes).at(n0, 0)};
  // Load l of the 2 C::loads of stage s into buf; past the last stage the range
  // is empty and zeros are written.
  constexpr int kLoads = 2 * C::loads;
  auto load = [&](u32x4* buf, idx_t s, int l) {
    const int op = l / C::loads, i = l % C::loads;
    const auto rs = buffer_rsrc(first[op], s < nk ? tile_bytes : 0);
    u32x4* to = buf + op * C::bm * CPR + i * C::threads + w * kWave;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        rs, (__attribute__((address_space(3))) void*)to, 16, (int)lane_off,
        (int)((uint32_t)s * C::bkb + (uint32_t)i * load_off), 0, 0);
  };

  // Fragment reads of step st from buf, kReads of them in the order the
  // matrix ops need them: every B fragment, then the A fragments.
  constexpr int kPer = LB / 16, kReads = P * (C::fm + C::fn);
  constexpr int kFragStride = 32 * CPR;
  auto read = [&](u32x4* buf, int st, int r, StepFrags<C>& f) {
    const int pl = r % P, k = r / P;
    const bool is_b = k < C::fn;
    const int frag = is_b ? k : k - C::fn;
    const int row = is_b ? C::bm + wn * C::wtn + col32 : wm * C::wtm + col32;
    const int ch = (pl * C::part + st * Mode::step_bytes + half * LB) / 16;
    const u32x4 v = (&rows_of(buf).at(row, ch))[frag * kFragStride];
    auto& to = is_b ? f.b[pl][frag] : f.a[pl][frag];
    if constexpr (LB == 16) {
      to = __builtin_bit_cast(mfma::bf16x8, v);
    } else {
      const u32x4 u = (&rows_of(buf).at(row, ch + 1))[frag * kFragStride];
      const auto both = __builtin_shufflevector(v, u, 0, 1, 2, 3, 4, 5, 6, 7);
      to = __builtin_bit_cast(mfma::i32x8, both);
    }
  };

  // the scales of this lane's rows and columns, loaded before the loop
  f32x4 sa[C::fm][4];
  float sb[C::fn];
  if constexpr (Mode::scaled) {
#pragma unroll
    for (int i = 0; i < C::fm; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        sa[i][q] = *(const f32x4*)&array(p.sa, 0)[m0 + wm * C::wtm + i * 32 + 8 * q + 4 * half];
#pragma unroll
    for (int j = 0; j < C::fn; ++j) sb[j] = array(p.sb, 0)[n0 + wn * C::wtn + j * 32 + col32];
  }

  mfma::f32x16 acc[C::fm][C::fn];
#pragma unroll
  for (int i = 0; i < C::fm; ++i)
#pragma unroll
    for (int j = 0; j < C::fn; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // Slots [o0, o1) of the 16 of one step: slot o is one matrix op on f (three
  // in the split mode), the reads of the next step's fragments that fall in it
  // (from `from`, step st, into g: kReads over the first kSpread slots) and,
  // unless kLoad0 is kNone, load o + kLoad0 of stage s into `to`.
  constexpr unsigned kMatrix = 0x008, kVmem = 0x010, kDsRead = 0x100;   // scheduling groups
  constexpr int kSlots = C::fm * C::fn, kNone = -100;
  static_assert(kLoads == kSlots, "one load a slot");
  auto slots = [&](auto first, auto last, auto spread, auto load0, const StepFrags<C>& f,
                   u32x4* from, int st, StepFrags<C>& g, u32x4* to, idx_t s) {
    constexpr int kSpread = spread, kLoad0 = load0;
#pragma unroll
    for (int o = first; o < last; ++o) {
      if (o < kSpread) {
#pragma unroll
        for (int r = o * kReads / kSpread; r < (o + 1) * kReads / kSpread; ++r) read(from, st, r, g);
      }
      if (kLoad0 != kNone && o + kLoad0 < kLoads) load(to, s, o + kLoad0);
      const int i = o / C::fn, j = o % C::fn;
      if constexpr (Mode::scaled) {
        acc[i][j] = mfma::fp8_32x32x64(f.a[0][i], f.b[0][j], acc[i][j]);
      } else {
        acc[i][j] = mfma::bf16_32x32x16(f.a[1][i], f.b[0][j], acc[i][j]);
        acc[i][j] = mfma::bf16_32x32x16(f.a[0][i], f.b[1][j], acc[i][j]);
        acc[i][j] = mfma::bf16_32x32x16(f.a[0][i], f.b[0][j], acc[i][j]);
      }
    }
#pragma unroll
    for (int o = first; o < last; ++o) {
      const int n = o < kSpread ? ((o + 1) * kReads / kSpread - o * kReads / kSpread) * kPer : 0;
      if (n == 1) __builtin_amdgcn_sched_group_barrier(kDsRead, 1, 0);
      if (n == 2) __builtin_amdgcn_sched_group_barrier(kDsRead, 2, 0);
      if (n == 4) __builtin_amdgcn_sched_group_barrier(kDsRead, 4, 0);
      if (kLoad0 != kNone && o + kLoad0 < kLoads) __builtin_amdgcn_sched_group_barrier(kVmem, 1, 0);
      __builtin_amdgcn_sched_group_barrier(kMatrix, Mode::scaled ? 1 : 3, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  StepFrags<C> f0, f1;
  // Stage s in cur, stage s + 1 on its way into next.  After kFree slots every
  // wave's reads of cur are done and the loads of stage s + 2 into it begin;
  // at the end of the first step stage s + 1 is complete: loads finish in
  // order, and kSlots - kFree younger ones may still be out.
  constexpr int kFree = 10, kYounger = kSlots - kFree;
  constexpr int kReadsDone = 0xC07F, kLoadsDone = 0x0F70 | kYounger;   // lgkmcnt(0), vmcnt
  auto stage = [&](u32x4* cur, u32x4* next, idx_t s) {
    slots(I<0>{}, I<kFree>{}, I<kSlots / 2>{}, I<kNone>{}, f0, cur, 1, f1, cur, s);
    __builtin_amdgcn_s_waitcnt(kReadsDone);
    bare_barrier();
    slots(I<kFree>{}, I<kSlots>{}, I<0>{}, I<-kFree>{}, f0, cur, 1, f1, cur, s + 2);
    __builtin_amdgcn_s_waitcnt(kLoadsDone);
    bare_barrier();
    slots(I<0>{}, I<kSlots>{}, I<kSlots>{}, I<kYounger>{}, f1, next, 0, f0, cur, s + 2);
  };
#pragma unroll
  for (int l = 0; l < kLoads; ++l) load(even, 0, l);
#pragma unroll
  for (int l = 0; l < kLoads; ++l) load(odd, 1, l);
  wait_stores();
  sync(thread);
#pragma unroll
  for (int r = 0; r < kReads; ++r) read(even, 0, r, f0);
  __builtin_amdgcn_sched_barrier(0);
#pragma clang loop unroll(disable)
  for (idx_t s = 0; s < nk; s += 2) {
    stage(even, odd, s);
    stage(odd, even, s + 1);   // zeros where the number of stages is odd
  }
  wait_stores();   // no load may write LDS after the block's end

  // C, one fragment row of 16 x fn stores at a time: a buffer range over the
  // tile's valid part of C drops what lies outside it, so every store is
  // unconditional, at a lane offset plus one uniform offset.
  const int32_t rows = (int32_t)(p.M - m0 < C::bm ? p.M - m0 : C::bm);
  const int32_t cols = (int32_t)(p.N - n0 < C::bn ? p.N - n0 : C::bn);
  const BufferWindow<4> win{(uint32_t)p.ldc, rows, cols};
  const auto rc = buffer_rsrc(&matrix(p.C, p.M, p.ldc).at(m0, n0), win.bytes());
  uint32_t at[C::fn];
#pragma unroll
  for (int j = 0; j < C::fn; ++j)
    at[j] = win.row(4 * half) + win.col(wn * C::wtn + j * 32 + col32);
#pragma unroll
  for (int i = 0; i < C::fm; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const uint32_t r0 = win.row(wm * C::wtm + i * 32 + mfma::acc_row(r, 0));
#pragma unroll
      for (int j = 0; j < C::fn; ++j) {
        float v = acc[i][j][r];
        if constexpr (Mode::scaled) v = (v * sa[i][r / 4][r % 4]) * sb[j];
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rc, (int)(at[j] + r0), 0, kNt ? 2 : 0);
      }
    }
}

}  // namespace gemm_nt
}  // namespace desc
