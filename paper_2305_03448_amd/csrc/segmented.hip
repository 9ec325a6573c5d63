// segmented.hip -- reduce and inclusive scan restarted at every segment
// (the batched form of the Sec. 5 reduction and scan): segment s covers
// positions [offsets[s], offsets[s+1]) of one int32 array.
//
// Work is cut into units: segment s of length L_s gives ceil(L_s / UNIT)
// units of at most UNIT consecutive elements (an empty segment gives none);
// UNIT is 8K to 64K elements, picked per size class by the tuning table or from
// the mean segment length (below).
// A unit finds its segment by a search over the exclusive prefix of the unit
// counts (64 entries a step, or two where the segments are few), loads its elements with dword-aligned 16-byte loads (segments
// start anywhere), and
//   reduce: sums them in int64; a segment of one unit stores its sum, the
//           units of a longer one combine theirs (below);
//   scan:   publishes the unit aggregate, looks back over the earlier units
//           of the same segment only (the look-back of the plain scan,
//           stopped at the segment's first unit), and writes its part of the
//           segment's scan.
//
// Reduce, up to kSegLds segments (unless there are many short ones, below): one
// persistent launch.  Every block computes the unit
// prefix into its LDS (S + 1 int32) and then walks its own contiguous range
// of units in order, keeping running sums per segment, so it streams through
// contiguous memory and synchronises only where a segment ends.  A segment
// split between ranges is finished by the block holding its end, from the
// tail sums the earlier blocks publish (tagged with the call's generation,
// handover.hpp) when their ranges are done; those blocks have smaller
// indices and were dispatched first.  The last block waits for every tail,
// then clears the words the previous call left past this call's and
// advances the generation, as the plain scan does, so no word older than
// the previous call can match a later tag.
//
// Scan (and the other reduces, and the batched forms): a
// one-block plan kernel writes the unit prefix to the workspace (zeroing
// the reduce outputs of segments without exactly one unit, which the units
// then add to atomically; clearing the scan status words), and a main
// kernel runs one block per unit (launched for the bound S + n / UNIT units;
// blocks past the total return at once, and units are handed out in block
// order, so a unit waits only on units whose blocks are already running).
// With many short segments a block of that kernel takes one unit per wave.
//
// Integer addition is associative, so results are exact and independent of
// the order.
#include "common.hpp"
#include "handover.hpp"
#include "launch.hpp"
#include "layouts.hpp"
#include "tuning.hpp"
#include "view.hpp"
#include "wave.hpp"
#include "wave_search.hpp"

namespace desc {
namespace {

// A unit is kBlock threads x kRounds rounds x 4 int32.
template <int kBlock_, int kRounds_>
struct UnitCfg {
  static constexpr int block = kBlock_;
  static constexpr int rounds = kRounds_;
  static constexpr int waves = kBlock_ / kWave;
  static constexpr int unit = waves * kWave * 4 * kRounds_;   // int32 per unit
};
constexpr int kMinUnit = 8192;   // smallest unit of the configurations below
constexpr uint64_t kFlagAggregate = 1, kFlagPrefix = 2;
constexpr int64_t kSegLds = 8192;   // segments whose unit prefix a block keeps in LDS

struct SegWs {
  int64_t* total;        // number of units (two-launch form)
  int64_t* unit_start;   // S + 1 entries (two-launch form)
  uint64_t* status;      // one word per unit (scan)
  uint64_t* words;       // two tail words per block (persistent reduce)
};

template <class C>
__device__ __forceinline__ int64_t units_of(int64_t len) { return layout::seg_units(len, C::unit); }

// Offsets are read clamped to [0, n]: offsets that break the documented
// precondition (non-decreasing, within the array) give unspecified results
// but never an access outside the array.
__device__ __forceinline__ int64_t clampn(int64_t v, int64_t n) { return layout::seg_clamp(v, n); }

// One block of kPlanBlock threads, kPlanPer consecutive segments per thread:
// unit counts and their exclusive prefix over the segments, a chunk of
// kPlanBlock * kPlanPer segments per pass with a running carry; then per-op
// initialisation.  Reduce: the outputs of segments that do not have exactly
// one unit are zeroed (atomics add into them; an empty segment sums to 0).
// Scan: the look-back status words are cleared.
constexpr int kPlanBlock = 1024, kPlanPer = 4, kPlanWaves = kPlanBlock / kWave;

template <class C, bool kScan>
__global__ __launch_bounds__(kPlanBlock) void plan_kernel(const int64_t* __restrict__ offsets,
                                                          int64_t n, int64_t S,
                                                          int64_t* __restrict__ total,
                                                          int64_t* __restrict__ unit_start,
                                                          int64_t* __restrict__ red_out,
                                                          uint64_t* __restrict__ status,
                                                          int64_t max_units) {
  __shared__ int64_t s_wsum[kPlanWaves];
  __shared__ int64_t s_carry;
  auto thread = thread_x<kPlanBlock>();
  auto wv = wave_of_block<kPlanBlock>();
  auto lane = lane_of_wave();
  auto off = array(offsets, S + 1);
  auto us = array(unit_start, S + 1);
  if (thread.index() == 0) s_carry = 0;
  sync(thread);
  for (idx_t base = 0; base < S; base += kPlanBlock * kPlanPer) {
    const idx_t s0 = base + thread.index() * kPlanPer;
    int64_t u[kPlanPer];
    int64_t mine = 0;
#pragma unroll
    for (int j = 0; j < kPlanPer; ++j) {
      const idx_t s = s0 + j;
      const int64_t len = s < S ? clampn(off[s + 1], n) - clampn(off[s], n) : 0;
      u[j] = s < S ? units_of<C>(len > 0 ? len : 0) : 0;
      if constexpr (!kScan) {
        if (s < S && u[j] != 1) array(red_out, S)[s] = 0;
      }
      mine += u[j];
    }
    // block-wide exclusive prefix of the per-thread unit counts (int64)
    int64_t incl = mine;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const int64_t t = __shfl_up(incl, d, kWave);
      if ((int)lane.index() >= d) incl += t;
    }
    if (lane.index() == kWave - 1) s_wsum[wv.index()] = incl;
    sync(thread);
    int64_t before = s_carry;
    for (int w = 0; w < kPlanWaves; ++w) before += (w < wv.index()) ? s_wsum[w] : 0;
    int64_t at = before + incl - mine;
#pragma unroll
    for (int j = 0; j < kPlanPer; ++j) {
      if (s0 + j < S) us[s0 + j] = at;
      at += u[j];
    }
    sync(thread);
    if (thread.index() == kPlanBlock - 1) s_carry = before + incl;
    sync(thread);
  }
  if (thread.index() == 0) {
    us[S] = s_carry;
    total[0] = s_carry;
  }
  if constexpr (kScan) {
    auto st = array(status, max_units);
    for (idx_t i = thread.index(); i < max_units; i += kPlanBlock) st[i] = 0;
  }
}

struct UnitInfo {
  idx_t seg, j, begin, len;   // segment, unit index inside it, first position, length
  bool single;                // the segment has one unit only
};

// Unit u of this block, found by wave 0 and shared.  The 64-way search takes
// two or three rounds of parallel loads where a binary search takes a dependent
// load per step, 14 of them (8 us a block) at 16384 segments.  Of few segments
// the binary search is the faster one, since its position is uniform and its
// loads are scalar ones that hit the scalar cache: up to 16 segments, and up to
// 64 where the blocks come in many rounds (reduce of 64 rows of 4 M 181 against
// 184 us, scan 416 / 422; 1000 rows of 60000 60 against 56).  In a scan of
// 64 segments with one round of blocks its steps lie in the serial chain of the
// call (262144 elements 8.2 against 7.5 us, 4.2 M 12.9 / 12.2).
__device__ __forceinline__ bool scalar_search(int64_t S, int64_t units) {
  constexpr int64_t kFewSegments = 16, kSomeSegments = 64, kManyUnits = 4096;
  return S <= kFewSegments || (S <= kSomeSegments && units > kManyUnits);
}
template <class C>
__device__ __forceinline__ bool unit_info(const int64_t* offsets, const int64_t* unit_start,
                                          int64_t n, int64_t S, int64_t total, idx_t u,
                                          UnitInfo* out) {
  __shared__ int64_t s_info[5];
  auto thread = thread_x<C::block>();
  if (u >= total) return false;
  if (thread.index() < kWave) {
    const auto us = array(unit_start, S + 1);
    const idx_t seg = scalar_search(S, total) ? layout::seg_of_unit(us, S, u)
                                         : wave_owner(unit_start, S, u);
    const layout::SegUnit su =
        layout::seg_unit_of(array(offsets, S + 1), us, n, C::unit, u, seg);
    if (thread.index() == 0) {
      s_info[0] = su.seg; s_info[1] = su.j; s_info[2] = su.begin;
      s_info[3] = su.len; s_info[4] = su.single;
    }
  }
  sync(thread);
  *out = UnitInfo{s_info[0], s_info[1], s_info[2], s_info[3], s_info[4] != 0};
  return true;
}

// Every block's plan for the persistent forms: s_us[s] = units before
// segment s (exclusive prefix of the unit counts), s_us[S] = the total.
// The counts are computed with strided, independent loads of the offsets
// (in flight together), then thread t scans ceil(S / kThreads) consecutive
// counts in LDS, made odd so that the lanes' counts lie in different banks
// (at 8000 segments 256 threads would be 32 words apart, all in one: the plan
// took 50 of the 74 us of a reduce of 8.6 M elements).
template <int kThreads>
__device__ __forceinline__ int32_t lds_unit_plan(const int64_t* offsets, int64_t n, int64_t S,
                                                 int64_t unit, int32_t* s_us, int32_t* s_wsum) {
  auto thread = thread_x<kThreads>();
  auto wv = wave_of_block<kThreads>();
  auto lane = lane_of_wave();
  auto off = array(offsets, S + 1);
  auto us = array(s_us, S + 1);
  for (idx_t s = thread.index(); s < S; s += kThreads) {
    const int64_t len = layout::seg_clamp(off[s + 1], n) - layout::seg_clamp(off[s], n);
    us[s] = (int32_t)layout::seg_units(len, unit);
  }
  sync(thread);
  const idx_t per = ((S + kThreads - 1) / kThreads) | 1;
  const idx_t s0 = thread.index() * per, s1 = s0 + per < S ? s0 + per : S;
  int32_t mine = 0;
  for (idx_t s = s0; s < s1; ++s) mine += us[s];
  int32_t incl = mine;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const int32_t t = __shfl_up(incl, d, kWave);
    if ((int)lane.index() >= d) incl += t;
  }
  if (lane.index() == kWave - 1) s_wsum[wv.index()] = incl;
  sync(thread);
  int32_t at = incl - mine, total = 0;
  for (int w = 0; w < kThreads / kWave; ++w) {
    const int32_t v = s_wsum[w];
    at += w < (int)wv.index() ? v : 0;
    total += v;
  }
  for (idx_t s = s0; s < s1; ++s) {
    const int32_t c = us[s];
    us[s] = at;
    at += c;
  }
  if (thread.index() == 0) us[S] = total;
  sync(thread);
  return total;
}

// First element of round r of the wave of thread t (a uniform value).
template <class C>
__device__ __forceinline__ idx_t round_start(uint32_t t, int r) {
  return ((idx_t)__builtin_amdgcn_readfirstlane(t / kWave) * C::rounds + r) * 256;
}

// Elements at .. at + 3 of a run of len >= 4 elements, 0 past its end, by one
// unconditional 16-byte load: a group of four that would cross the end starts
// at the last four elements instead, whose first words belong to earlier
// groups and are dropped (with every word guarded, 16384 segments of 1000
// elements on average took 268 us to scan).
template <bool kNt>
__device__ __forceinline__ void load_group(const int32_t* run, int at, int len, uint32_t (&x)[4]) {
  const int from = at < len - 4 ? at : len - 4;
  const i32x4u* p = (const i32x4u*)(run + from);
  i32x4u q;
  if constexpr (kNt) q = __builtin_nontemporal_load(p);
  else q = *p;
  const int d = at - from;   // 0 but for the group that crosses the end and those past it
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    uint32_t v = (uint32_t)q[k];
    if (k < 3) v = d == 1 ? (uint32_t)q[k + 1] : v;
    if (k < 2) v = d == 2 ? (uint32_t)q[k + 2] : v;
    if (k < 1) v = d == 3 ? (uint32_t)q[k + 3] : v;
    x[k] = at + k < len ? v : 0u;
  }
}
// The up to three elements of a shorter run: thread 0's.
__device__ __forceinline__ void load_tiny(const int32_t* run, int len, bool first,
                                          uint32_t (&x)[4]) {
  if (!first) return;
#pragma unroll
  for (int k = 0; k < 3; ++k)
    if (k < len) x[k] = (uint32_t)run[k];
}

// The unit's elements as [waves][rounds][lanes][4]; x[r][k] gets element
// (w * rounds + r) * 256 + lane * 4 + k (0 beyond the unit's length).
// kNt: non-temporal 16-byte loads (the reduce, which only streams its input;
// 4 % faster there, 3 % slower for the scan, which writes as it reads).
template <class C, bool kNt = false>
__device__ __forceinline__ void load_unit(const int32_t* in, const UnitInfo& ui,
                                          uint32_t (&x)[C::rounds][4]) {
  constexpr int kWaves = C::waves, kRounds = C::rounds, kUnit = C::unit;
  const uint32_t t = opaque_thread();
  const Wave<kWaves> wv{(idx_t)(t / kWave), kWaves};
  const Lane<kWave> lane{(idx_t)(t % kWave), kWave};
  auto unit = array(in, 0).snd(ui.begin);
  if (ui.len == kUnit) {
    auto mine = layout::wave_striped<kWaves, kRounds>(array((const i32x4u*)&unit[0], kUnit / 4),
                                                      0, wv, lane);
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      i32x4u q;
      if constexpr (kNt) q = __builtin_nontemporal_load(&mine[r]);
      else q = mine[r];
      x[r][0] = (uint32_t)q.x; x[r][1] = (uint32_t)q.y;
      x[r][2] = (uint32_t)q.z; x[r][3] = (uint32_t)q.w;
    }
  } else {
    // a partial unit; a wave whose rounds all lie past the end loads nothing
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
#pragma unroll
      for (int k = 0; k < 4; ++k) x[r][k] = 0u;
    const int len = (int)ui.len;
    if (len < 4) {
      load_tiny(&unit[0], len, t == 0, x[0]);
    } else if (round_start<C>(t, 0) < ui.len) {
      auto mine = layout::wave_striped<kWaves, kRounds>(array(&unit[0], kUnit).group<4>(), 0, wv,
                                                        lane);
#pragma unroll
      for (int r = 0; r < kRounds; ++r)
        load_group<kNt>(&unit[0], (int)mine.idx(r).pos(0), len, x[r]);
    }
  }
}

// The unit's sum (int64), valid in thread 0.
template <class C>
__device__ __forceinline__ int64_t reduce_unit(const int32_t* in, const UnitInfo& ui,
                                               int64_t* s_w) {
  constexpr int kBlock = C::block, kWaves = C::waves, kRounds = C::rounds;
  auto thread = thread_x<kBlock>();
  auto wv = wave_of_block<kBlock>();
  uint32_t x[kRounds][4];
  load_unit<C, true>(in, ui, x);
  int64_t acc = 0;
#pragma unroll
  for (int r = 0; r < kRounds; ++r)
#pragma unroll
    for (int k = 0; k < 4; ++k) acc += (int64_t)(int32_t)x[r][k];
  acc = wave::sum_i64(acc);
  if (lane_of_wave().index() == 0) s_w[wv.index()] = acc;
  sync(thread);
  int64_t t = 0;
  if (thread.index() == 0) {
#pragma unroll
    for (int w = 0; w < kWaves; ++w) t += s_w[w];
  }
  return t;
}

template <class C>
__global__ __launch_bounds__(C::block) void seg_reduce_kernel(const int32_t* __restrict__ in,
                                                            int64_t n,
                                                            const int64_t* __restrict__ offsets,
                                                            int64_t S,
                                                            const int64_t* __restrict__ total,
                                                            const int64_t* __restrict__ unit_start,
                                                            int64_t* __restrict__ out,
                                                            int64_t block0) {
  __shared__ int64_t s_w[C::waves];
  UnitInfo ui;
  if (!unit_info<C>(offsets, unit_start, n, S, total[0], block0 + block_x().index(), &ui)) return;
  const int64_t t = reduce_unit<C>(in, ui, s_w);
  if (thread_x<C::block>().index() == 0) {
    auto o = array(out, S);
    if (ui.single) o[ui.seg] = t;
    else __hip_atomic_fetch_add(&o[ui.seg], t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// The persistent reduce (up to kSegLds segments): see the file comment.
// Block b takes the contiguous units [T b / G, T (b + 1) / G) and walks
// them in order, each thread adding its elements into a running int64 sum
// for the current segment; at the end of a segment (or of the range) the
// block adds the threads' sums.  A segment that starts and ends in the range
// is stored at once.  The range's last segment, when it continues past the
// range, is the block's tail: its part is published (every block publishes
// one tail word pair, 0 when it has none).  The range's first segment, when
// it started in an earlier range and ends in this one, is resolved at the
// end: its part here plus the tails of the earlier blocks back to the one
// where it starts -- blocks of smaller index, dispatched earlier, which
// publish once their ranges are done.  Block G - 1 ends the call.
template <class C>
__global__ __launch_bounds__(C::block) void seg_reduce_persistent_kernel(
    const int32_t* __restrict__ in, int64_t n, const int64_t* __restrict__ offsets, int64_t S,
    int64_t* __restrict__ out, uint64_t* __restrict__ words, WsHeader* __restrict__ hdr) {
  constexpr int kRounds = C::rounds;
  __shared__ int32_t s_us[kSegLds + 1];
  __shared__ int32_t s_wsum[C::waves];
  __shared__ int64_t s_w[C::waves];
  __shared__ CallState s_call;
  auto block = block_x();
  auto thread = thread_x<C::block>();
  auto wv = wave_of_block<C::block>();
  if (thread.index() == 0) s_call = read_call_state(hdr);
  const int32_t T = lds_unit_plan<C::block>(offsets, n, S, C::unit, s_us, s_wsum);  // syncs
  const uint32_t gen = s_call.gen;
  const uint64_t tag = handover::tag_of(gen);
  const idx_t G = block.count(), b = block.index();
  auto first_unit = [&](idx_t k) { return (idx_t)((int64_t)T * k / G); };
  const idx_t u0 = first_unit(b), u1 = first_unit(b + 1);
  auto o = array(out, S);
  auto off = array(offsets, S + 1);
  auto us = array(s_us, S + 1);
  auto tails = array(words, 2 * G).group<2>();              // [G][2]
  for (idx_t s = b * C::block + thread.index(); s < S; s += G * C::block)
    if (us[s] == us[s + 1]) o[s] = 0;                       // empty segment
  // the threads' sums added over the block, valid in thread 0
  auto block_total = [&](int64_t v) {
    v = wave::sum_i64(v);
    sync(thread);                                           // earlier readers of s_w are done
    if (lane_of_wave().index() == 0) s_w[wv.index()] = v;
    sync(thread);
    int64_t t = 0;
    if (thread.index() == 0)
      for (int w = 0; w < C::waves; ++w) t += s_w[w];
    return t;
  };
  int64_t tail = 0, head = 0;
  idx_t head_seg = -1;
  int64_t acc = 0;
  idx_t seg = u0 < u1 ? layout::seg_of_unit(us, S, u0) : 0;
  int64_t sb = layout::seg_clamp(off[seg], n), se = layout::seg_clamp(off[seg + 1], n);
#pragma clang loop unroll(disable)
  for (idx_t u = u0; u < u1; ++u) {
    if (us[seg + 1] <= u) {                                  // the next non-empty segment
      do ++seg; while (us[seg + 1] <= u);
      sb = layout::seg_clamp(off[seg], n);
      se = layout::seg_clamp(off[seg + 1], n);
    }
    const idx_t j = u - us[seg], begin = sb + j * C::unit;
    const UnitInfo ui{seg, j, begin, se - begin < C::unit ? se - begin : C::unit, false};
    uint32_t x[kRounds][4];
    load_unit<C, true>(in, ui, x);
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
#pragma unroll
      for (int k = 0; k < 4; ++k) acc += (int64_t)(int32_t)x[r][k];
    if (u + 1 == us[seg + 1] || u + 1 == u1) {               // the segment's part here ends
      const int64_t total = block_total(acc);
      acc = 0;
      if (thread.index() == 0) {
        if (us[seg + 1] > u1) tail = total;                  // continues past the range
        else if (us[seg] < u0) { head = total; head_seg = seg; }
        else o[seg] = total;
      }
    }
  }
  if (thread.index() == 0) {
    handover::publish(&tails.idx(b)[0], tag, (uint64_t)tail);
    if (head_seg >= 0) {                                     // add the earlier blocks' tails
      bool ok = true;
      for (idx_t k = b - 1; k >= 0; --k) {
        if (first_unit(k) == first_unit(k + 1)) continue;   // an empty range
        uint64_t v = 0;
        ok = handover::poll(&tails.idx(k)[0], tag, v, s_call.polls) && ok;
        head += (int64_t)v;
        if (first_unit(k) <= us[head_seg]) break;            // the block where it starts
      }
      if (!ok) set_error(hdr, kDevWaitLimit);
      o[head_seg] = head;
    }
  }
  if (b == G - 1) {
    // every block publishes its tail after reading the generation: once all
    // have, advance it and clear what the previous call left past 2 G words
    sync(thread);
    bool ok = true;
    for (idx_t k = thread.index(); k < G; k += C::block) {
      uint64_t v = 0;
      ok = handover::poll(&tails.idx(k)[0], tag, v, s_call.polls) && ok;
    }
    if (!ok) set_error(hdr, kDevWaitLimit);
    sync(thread);
    const uint64_t used = 2 * (uint64_t)G;
    const uint64_t hw = __hip_atomic_load(&hdr->hw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    clear_words<C::block>(words, used, hw, thread.index());
    if (thread.index() == 0) {
      __hip_atomic_store(&hdr->hw, used, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      store_u32(&hdr->gen, next_gen(gen));
    }
  }
}

__device__ __forceinline__ uint64_t pack(uint64_t flag, uint32_t v) { return (flag << 62) | v; }

// Exclusive prefix of unit u from the earlier units of its segment
// (j of them, layout::lookback_unit's windows); one whole wave.
// At most `max_polls` polls (none with max_polls = 0); a wait that runs out
// records kDevWaitLimit and returns the partial prefix.
__device__ __forceinline__ uint32_t seg_look_back(const uint64_t* status, idx_t u, idx_t j,
                                                  uint32_t max_polls, WsHeader* hdr) {
  const int lane = wave::lane_id();
  uint32_t excl = 0;
  auto st = array(status, u);
  idx_t window = 0;
  for (uint32_t polls = 0; kWave * window < j; ++polls) {
    if (polls == max_polls) {
      if (lane == 0) set_error(hdr, kDevWaitLimit);
      break;
    }
    const bool in_seg = layout::lookback_in_segment(j, window, lane);
    const uint64_t w =
        in_seg ? load_status(&st[layout::lookback_unit(u, window, lane)]) : pack(kFlagPrefix, 0u);
    const uint32_t flag = (uint32_t)(w >> 62);
    const uint64_t pmask = __ballot(flag == kFlagPrefix && in_seg);
    const idx_t left = j - kWave * window;
    const int width = left < kWave ? (int)left : kWave;
    const int first_p = pmask ? __builtin_ctzll(pmask) : width - 1;
    const uint64_t need = first_p == 63 ? ~0ull : ((2ull << first_p) - 1);
    if (__ballot(flag == 0 && in_seg) & need) {
      __builtin_amdgcn_s_sleep(2);
      continue;
    }
    excl += wave::sum_u32(lane <= first_p && in_seg ? (uint32_t)w : 0u);
    if (pmask) break;
    ++window;
  }
  return excl;
}

struct ScanShared {
  uint32_t wtot[16];   // wave totals (up to 1024 threads)
  uint32_t prefix;     // the unit's exclusive prefix
};

// A wave's part of a unit scanned in registers, from its first element on.
template <class C>
__device__ __forceinline__ void scan_wave(uint32_t (&x)[C::rounds][4]) {
  constexpr int kRounds = C::rounds;
  uint32_t carry = 0;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    x[r][1] += x[r][0];
    x[r][2] += x[r][1];
    x[r][3] += x[r][2];
    const uint32_t incl = wave::inclusive_add_u32(x[r][3]);
    const uint32_t ex = carry + incl - x[r][3];
#pragma unroll
    for (int k = 0; k < 4; ++k) x[r][k] += ex;
    carry += wave::lane_read_u32(incl, kWave - 1);
  }
}

// Those values, `add` before each, to the unit's positions of `out`.
template <class C>
__device__ __forceinline__ void store_unit(int32_t* __restrict__ out, const UnitInfo& ui,
                                           const uint32_t (&x)[C::rounds][4], uint32_t add) {
  constexpr int kWaves = C::waves, kRounds = C::rounds, kUnit = C::unit;
  auto unit = array(out, 0).snd(ui.begin);
  const uint32_t ot = opaque_thread();
  const Wave<kWaves> owv{(idx_t)(ot / kWave), kWaves};
  const Lane<kWave> olane{(idx_t)(ot % kWave), kWave};
  if (ui.len == kUnit) {
    auto mine = layout::wave_striped<kWaves, kRounds>(array((i32x4u*)&unit[0], kUnit / 4), 0,
                                                      owv, olane);
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      i32x4u q;
      q.x = (int32_t)(x[r][0] + add); q.y = (int32_t)(x[r][1] + add);
      q.z = (int32_t)(x[r][2] + add); q.w = (int32_t)(x[r][3] + add);
      mine[r] = q;
    }
  } else {                                   // as the loads of a partial unit
    auto vec = layout::wave_striped<kWaves, kRounds>(array((i32x4u*)&unit[0], kUnit / 4), 0, owv,
                                                     olane);
    auto mine = layout::wave_striped<kWaves, kRounds>(array(&unit[0], kUnit).group<4>(), 0,
                                                      owv, olane);
    const idx_t left = ui.len - round_start<C>(ot, 0);
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      if (256 * (r + 1) <= left) {
        i32x4u q;
        q.x = (int32_t)(x[r][0] + add); q.y = (int32_t)(x[r][1] + add);
        q.z = (int32_t)(x[r][2] + add); q.w = (int32_t)(x[r][3] + add);
        vec[r] = q;
      } else if (256 * r < left) {
        auto g = mine.idx(r);
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (g.pos(k) < ui.len) g[k] = (int32_t)(x[r][k] + add);
      }
    }
  }
}

// One unit of the segmented scan (u its index).
template <class C>
__device__ __forceinline__ void scan_unit(const int32_t* __restrict__ in,
                                          int32_t* __restrict__ out, const UnitInfo& ui, idx_t u,
                                          uint64_t* __restrict__ status, uint32_t polls,
                                          WsHeader* __restrict__ hdr, ScanShared& sh) {
  constexpr int kBlock = C::block, kWaves = C::waves, kRounds = C::rounds;
  static_assert(kWaves <= 16, "wave totals fit ScanShared");
  auto thread = thread_x<kBlock>();
  auto wv = wave_of_block<kBlock>();
  auto lane = lane_of_wave();
  uint32_t x[kRounds][4];
  load_unit<C>(in, ui, x);

  uint32_t lsum = 0;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) lsum += x[r][0] + x[r][1] + x[r][2] + x[r][3];
  const uint32_t wsum = wave::sum_u32(lsum);
  if (lane.index() == 0) sh.wtot[wv.index()] = wsum;
  sync(thread);
  uint32_t wex = 0, agg = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const uint32_t v = sh.wtot[w];
    wex += (w < wv.index()) ? v : 0u;
    agg += v;
  }
  auto st = array(status, u + 1);
  if (wv.index() == 0) {
    uint32_t excl = 0;
    if (ui.j == 0) {
      if (lane.index() == 0) store_status(&st[u], pack(kFlagPrefix, agg));
    } else {
      if (lane.index() == 0) store_status(&st[u], pack(kFlagAggregate, agg));
      excl = seg_look_back(status, u, ui.j, polls, hdr);
      if (lane.index() == 0) store_status(&st[u], pack(kFlagPrefix, excl + agg));
    }
    if (lane.index() == 0) sh.prefix = excl;
  }
  scan_wave<C>(x);
  sync(thread);
  const uint32_t add = sh.prefix + wex;
  store_unit<C>(out, ui, x, add);
}

// Eight rounds take 64 registers, which is two blocks of 1024 threads on a CU.
template <class C>
__global__ __launch_bounds__(C::block) __attribute__((amdgpu_waves_per_eu(C::rounds == 8 ? 8 : 1)))
void seg_scan_kernel(const int32_t* __restrict__ in, int32_t* __restrict__ out, int64_t n,
                     const int64_t* __restrict__ offsets, int64_t S,
                     const int64_t* __restrict__ total, const int64_t* __restrict__ unit_start,
                     uint64_t* __restrict__ status, WsHeader* __restrict__ hdr, int64_t block0) {
  __shared__ ScanShared sh;
  UnitInfo ui;
  const idx_t u = block0 + block_x().index();
  if (!unit_info<C>(offsets, unit_start, n, S, total[0], u, &ui)) return;
  scan_unit<C>(in, out, ui, u, status,
               max_polls(__hip_atomic_load(&hdr->wait_limit, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT)),
               hdr, sh);
}

// --------------------------------------------------------------------------
// Many short segments.  With a block per unit, a segment of tens of elements
// still costs a block its chain of loads (total, search, offsets, values:
// about 4 us with 8 blocks a CU, 50-60 us for 16384 segments).  Here a block
// takes one unit per wave: the waves look their units up side by side, each
// wave whose unit is a whole segment of at most kShortLen elements reduces or
// scans it alone, and then the block works through its other units.  A reduce
// takes them in order, as a block per unit would.  A scan may not where a
// segment has several units: a unit published after an earlier one's look-back
// would make every block wait for the one before it (one segment of 4 M
// elements among 4095 short ones: 891 us, 27 with a block per unit; of 20 M
// among 16383: 4440 and 287).  Then the block first publishes the sums of all its
// units, looks back once, and reads the units again to write them (21 and 57 us).
constexpr int kShortRounds = 4;
constexpr int kShortLen = 256 * kShortRounds;

// A short segment's values: round r of lane l holds elements 256 r + 4 l ...
__device__ __forceinline__ void load_short(const int32_t* in, idx_t begin, int len,
                                           uint32_t (&x)[kShortRounds][4]) {
  auto run = array(in, 0).snd(begin);
  auto mine = layout::wave_striped<1, kShortRounds>(array(&run[0], kShortLen).group<4>(), 0,
                                                    Wave<1>{0, 1}, lane_of_wave());
#pragma unroll
  for (int r = 0; r < kShortRounds; ++r)
#pragma unroll
    for (int k = 0; k < 4; ++k) x[r][k] = 0u;
  if (len < 4) {
    load_tiny(&run[0], len, lane_of_wave().index() == 0, x[0]);
    return;
  }
#pragma unroll
  for (int r = 0; r < kShortRounds; ++r)
    if (256 * r < len) load_group<false>(&run[0], (int)mine.idx(r).pos(0), len, x[r]);
}

// The partial sums of a block's units, by unit and wave, and their prefixes.
template <class C>
struct RunShared {
  uint32_t part[C::waves][C::waves];
  uint32_t prefix[C::waves];
};

// This block's units, one per wave, in LDS.
constexpr uint8_t kShortUnit = 0, kWholeUnit = 1, kRunUnit = 2;   // kRunUnit: others wait for it
template <class C>
struct BlockUnits {
  UnitInfo ui[C::waves];
  int count;
  __attribute__((aligned(4))) uint8_t kind[C::waves];
  // Whether some unit is not a short one, and whether one past the first is a
  // kRunUnit: a word read for four units.
  __device__ bool any_long() const { return kinds(0x03030303u, 0x03030303u); }
  __device__ bool any_run() const { return kinds(0x02020200u, 0x02020202u); }
  __device__ bool kinds(uint32_t first, uint32_t others) const {
    const uint32_t* k = (const uint32_t*)kind;
    uint32_t found = k[0] & first;
#pragma unroll
    for (int i = 1; i < C::waves / 4; ++i) found |= k[i] & others;
    return found != 0;
  }
};
__device__ __forceinline__ bool is_short(const UnitInfo& ui) {
  return ui.single && ui.len <= kShortLen;
}
template <class C>
__device__ __forceinline__ void find_units(const int64_t* offsets, const int64_t* unit_start,
                                           int64_t n, int64_t S, layout::BlockRange mine,
                                           BlockUnits<C>& bu) {
  auto thread = thread_x<C::block>();
  const int w = (int)wave_of_block<C::block>().index();
  if (w < mine.count) {
    const idx_t u = mine.first + w;
    const layout::SegUnit su =
        layout::seg_unit_of(array(offsets, S + 1), array(unit_start, S + 1), n, C::unit, u,
                            wave_owner(unit_start, S, u));
    const UnitInfo ui{su.seg, su.j, su.begin, su.len, su.single};
    if (lane_of_wave().index() == 0) {
      bu.ui[w] = ui;
      bu.kind[w] = is_short(ui) ? kShortUnit : ui.single ? kWholeUnit : kRunUnit;
    }
  } else if (lane_of_wave().index() == 0) {
    bu.kind[w] = kShortUnit;
  }
  if (thread.index() == 0) bu.count = mine.count;
  sync(thread);
}

// The block's units but the short ones (the first is unit u0), with one
// look-back: only the first unit can have its predecessor in another block.
template <class C>
__device__ __forceinline__ void scan_run(const int32_t* __restrict__ in, int32_t* __restrict__ out,
                                         const BlockUnits<C>& bu, idx_t u0,
                                         uint64_t* __restrict__ status, uint32_t polls,
                                         WsHeader* __restrict__ hdr, RunShared<C>& sh) {
  constexpr int kWaves = C::waves, kRounds = C::rounds;
  auto thread = thread_x<C::block>();
  const int w = (int)wave_of_block<C::block>().index(), lane = (int)lane_of_wave().index();
#pragma clang loop unroll(disable)
  for (int i = 0; i < bu.count; ++i) {
    if (bu.kind[i] == kShortUnit) continue;
    uint32_t x[kRounds][4];
    load_unit<C>(in, bu.ui[i], x);
    uint32_t sum = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) sum += x[r][0] + x[r][1] + x[r][2] + x[r][3];
    sum = wave::sum_u32(sum);
    if (lane == 0) sh.part[i][w] = sum;
  }
  sync(thread);
  if (w == 0) {                               // lane i: unit i
    auto st = array(status, u0 + bu.count);
    const bool mine = lane < bu.count && bu.kind[lane] != kShortUnit;
    const idx_t j = mine ? bu.ui[lane].j : 0;
    uint32_t sum = 0;
    if (mine) {
#pragma unroll
      for (int v = 0; v < kWaves; ++v) sum += sh.part[lane][v];
      store_status(&st[u0 + lane], pack(j == 0 ? kFlagPrefix : kFlagAggregate, sum));
    }
    uint32_t before = bu.ui[0].j > 0 ? seg_look_back(status, u0, bu.ui[0].j, polls, hdr) : 0u;
    uint32_t excl = 0;
    for (int i = 0; i < bu.count; ++i) {
      if (bu.ui[i].j == 0) before = 0;
      if (lane == i) excl = before;
      before += wave::lane_read_u32(sum, i);
    }
    if (mine) {
      if (j > 0) store_status(&st[u0 + lane], pack(kFlagPrefix, excl + sum));
      sh.prefix[lane] = excl;
    }
  }
  sync(thread);
#pragma clang loop unroll(disable)
  for (int i = 0; i < bu.count; ++i) {
    if (bu.kind[i] == kShortUnit) continue;
    uint32_t x[kRounds][4];
    load_unit<C>(in, bu.ui[i], x);
    uint32_t add = sh.prefix[i];
#pragma unroll
    for (int v = 0; v < kWaves; ++v) add += v < w ? sh.part[i][v] : 0u;
    scan_wave<C>(x);
    store_unit<C>(out, bu.ui[i], x, add);
  }
}

template <class C>
__global__ __launch_bounds__(C::block) void seg_reduce_short_kernel(
    const int32_t* __restrict__ in, int64_t n, const int64_t* __restrict__ offsets, int64_t S,
    const int64_t* __restrict__ total, int64_t max_units, const int64_t* __restrict__ unit_start,
    int64_t* __restrict__ out, int64_t block0) {
  __shared__ BlockUnits<C> bu;
  __shared__ int64_t s_w[C::waves];
  const auto mine = layout::block_units<C::waves>(block0 + block_x().index(), total[0], max_units);
  if (mine.count <= 0) return;
  find_units<C>(offsets, unit_start, n, S, mine, bu);
  auto thread = thread_x<C::block>();
  auto o = array(out, S);
  const int w = (int)wave_of_block<C::block>().index();
  if (w < mine.count && bu.kind[w] == kShortUnit) {
    uint32_t x[kShortRounds][4];
    load_short(in, bu.ui[w].begin, (int)bu.ui[w].len, x);
    int64_t acc = 0;
#pragma unroll
    for (int r = 0; r < kShortRounds; ++r)
#pragma unroll
      for (int k = 0; k < 4; ++k) acc += (int64_t)(int32_t)x[r][k];
    acc = wave::sum_i64(acc);
    if (lane_of_wave().index() == 0) o[bu.ui[w].seg] = acc;
  }
  if (!bu.any_long()) return;
#pragma clang loop unroll(disable)
  for (int i = 0; i < bu.count; ++i) {
    if (bu.kind[i] == kShortUnit) continue;
    const int64_t t = reduce_unit<C>(in, bu.ui[i], s_w);
    if (thread.index() == 0) {
      if (bu.ui[i].single) o[bu.ui[i].seg] = t;
      else __hip_atomic_fetch_add(&o[bu.ui[i].seg], t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    sync(thread);                          // s_w is reused by the next unit
  }
}

template <class C>
__global__ __launch_bounds__(C::block) void seg_scan_short_kernel(
    const int32_t* __restrict__ in, int32_t* __restrict__ out, int64_t n,
    const int64_t* __restrict__ offsets, int64_t S, const int64_t* __restrict__ total,
    int64_t max_units, const int64_t* __restrict__ unit_start, uint64_t* __restrict__ status,
    WsHeader* __restrict__ hdr, int64_t block0) {
  __shared__ BlockUnits<C> bu;
  __shared__ union {
    ScanShared one;
    RunShared<C> run;
  } sh;
  const auto mine = layout::block_units<C::waves>(block0 + block_x().index(), total[0], max_units);
  if (mine.count <= 0) return;
  find_units<C>(offsets, unit_start, n, S, mine, bu);
  auto thread = thread_x<C::block>();
  const int w = (int)wave_of_block<C::block>().index();
  if (w < mine.count && bu.kind[w] == kShortUnit) {   // whole segments: nothing to publish or look up
    const idx_t len = bu.ui[w].len;
    uint32_t x[kShortRounds][4];
    load_short(in, bu.ui[w].begin, (int)len, x);
    auto run = array(out, 0).snd(bu.ui[w].begin);
    auto groups = layout::wave_striped<1, kShortRounds>(
        array(&run[0], kShortLen).template group<4>(), 0, Wave<1>{0, 1}, lane_of_wave());
    uint32_t carry = 0;
#pragma unroll
    for (int r = 0; r < kShortRounds; ++r) {
      x[r][1] += x[r][0];
      x[r][2] += x[r][1];
      x[r][3] += x[r][2];
      const uint32_t incl = wave::inclusive_add_u32(x[r][3]);
      const uint32_t ex = carry + incl - x[r][3];
      auto g = groups.idx(r);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (g.pos(k) < len) g[k] = (int32_t)(x[r][k] + ex);
      carry += wave::lane_read_u32(incl, kWave - 1);
    }
  }
  if (!bu.any_long()) return;
  const uint32_t polls = max_polls(
      __hip_atomic_load(&hdr->wait_limit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  if (bu.any_run()) {
    scan_run<C>(in, out, bu, mine.first, status, polls, hdr, sh.run);
    return;
  }
#pragma clang loop unroll(disable)
  for (int i = 0; i < bu.count; ++i) {
    if (bu.kind[i] == kShortUnit) continue;
    scan_unit<C>(in, out, bu.ui[i], mine.first + i, status, polls, hdr, sh.one);
    sync(thread);                          // sh is reused by the next unit
  }
}

// Upper bound on the units of any configuration (the smallest unit).
int64_t max_units(int64_t n, int64_t S) { return S + (n + kMinUnit - 1) / kMinUnit; }
int64_t round64(int64_t b) { return (b + 63) & ~(int64_t)63; }

// Workspace: header; the unit total of the two-launch form (one 64-byte
// line); the state words at a fixed place, so that the extent a call leaves
// in the header (hw) means the same words to the next call whatever its
// size -- for the scan the status words (one per unit, both forms), for the
// reduce the persistent form's tail words (two per block); then
// the two-launch form's unit prefix (S + 1 int64), whose values (below
// 2^31) never carry a tag or a flag if a later call finds them among its
// state words.
constexpr int64_t kMaxReduceBlocks = 4096;   // grid of the persistent reduce, at most
int64_t state_words(int64_t n, int64_t S, bool scan) {
  const int64_t mu = max_units(n, S);
  return scan ? mu : 2 * (mu < kMaxReduceBlocks ? mu : kMaxReduceBlocks);
}

SegWs carve(void* ws, int64_t n, int64_t S, bool scan) {
  uint8_t* w = (uint8_t*)ws;
  SegWs r;
  r.total = (int64_t*)(w + sizeof(WsHeader));
  r.status = (uint64_t*)(w + sizeof(WsHeader) + 64);
  r.words = r.status;
  r.unit_start = (int64_t*)(w + sizeof(WsHeader) + 64 + round64(state_words(n, S, scan) * 8));
  return r;
}

// The persistent forms: up to kSegLds segments and unit counts in int32.
bool persistent_fits(int64_t n, int64_t S) {
  return S > 0 && S <= kSegLds && max_units(n, S) < (1ll << 31);
}

// Whether a call takes the form for many short segments (lengths log-uniform,
// so that half of them are far below the mean; us, one unit per block or the
// persistent reduce / this form):
//   reduce, mean length   380: 4000 segments 19 / 13, 8192: 33 / 20, 16384: 51 / 32
//                        2900: 4000 segments 24 / 20, 8192: 42 / 33, 16384: 73 / 56
//                         23K: 2048 segments 42 / 40, 8192: 145 / 131, 16384: 273 / 257
//     and below 2000 segments within 1 us either way; of 74K, where the
//     persistent reduce is as fast (8192: 371 / 367) and a block per unit is
//     not (9000: 435 / 410);
//   scan, mean length     380: 2048 segments 11.8 / 14.4, 4096: 17.6 / 15.9, 8192: 30 / 24
//                        1000: 2048 segments 13 / 17, 4096: 19 / 20, 6000: 27 / 25, 8192: 33 / 29
//                        1370: 2048 segments 15 / 18, 4096: 21 / 22, 6000: 28.0 / 28.1,
//                              8192: 35 / 34, 16384: 61 / 55
//                        2900: 4000 segments 27 / 37, 16384: 99 / 112
//     since the units of long segments in one block follow each other where
//     separate blocks overlap them.  Lengths all alike above 1024, the longest
//     segment of a wave, are its worst case (1030: 2048 segments 12 / 17, 6000
//     26 / 28, 16384 57 / 57), and its best below (2048 of 500: 9).
constexpr int64_t kShortCount = 2048, kShortReduceMean = 32768;
constexpr int64_t kManyShort = 6000, kShortScanMean = 1024, kManyShortScanMean = 1536;
bool short_reduce(int64_t n, int64_t S, bool persistent) {
  return S >= kShortCount && (n <= kShortReduceMean * S || !persistent);
}
bool short_scan(int64_t n, int64_t S) {
  return S >= kShortCount && n <= (S < kManyShort ? kShortScanMean : kManyShortScanMean) * S;
}

// Unit size by mean length ("by_mean"; us, units of 8K / 16K / 32K): a unit
// shorter than the segments splits them into more units to look back over,
// a longer one leaves most of a block idle on the segments it covers.
//   reduce  16384 segments of 2900 on average: 73 / 106 / 221; 8192 of 23K:
//           145 / 143 / 163; 4096 of 76K (persistent): 208 / 206 / 195; 9000
//           of 74K (a wave's unit each): 430 / 410 / 463
//   scan    16384 of 8.7K: 226 / 231 / 319; 8192 of 23K: 301 / 288 / 299;
//           1000 of 78K: 148 / 131 / 125; 4096 of 76K: 553 / 475 / 450
// Up to 384 units of 8K in all (1.5 a CU) the scan takes those whatever the
// mean, or it leaves CUs idle: one segment of 262144 7.5 / 8.4 / 9.3, two of 1.5 M
// 11.2 / 11.5 / 12.0, 30 of 100K 10.6 / 11.3 / 12.4; of 6 M in all 18.7 / 17.5 / 16.4 as
// one segment, 14.2 / 14.9 / 14.7 as 30.  Not the reduce, where the block that
// ends a segment adds up the tails of all before it: one segment of 262144
// 16.7 / 10.8 / 8.4, of 4 M 211 / 105 / 57.
constexpr int64_t kUnit8Reduce = 32768, kUnit8Scan = 12288, kUnit16Scan = 49152;
constexpr int64_t kFewUnitsScan = 384 * 8192;
int reduce_by_mean(int64_t n, int64_t S, bool persistent) {
  if (n <= kUnit8Reduce * S) return 0;
  return short_reduce(n, S, persistent) ? 1 : 2;
}
int scan_by_mean(int64_t n, int64_t S) {
  if (n <= kUnit8Scan * S || n <= kFewUnitsScan) return 0;
  return n <= kUnit16Scan * S ? 1 : 2;
}

// `blocks` blocks in as many launches as one grid's count of threads asks for
// (one below 2^22 blocks); a unit waits only for units of earlier blocks, so of
// this launch or one before it.
template <class C, class F>
hipError_t in_grids(int64_t blocks, F&& launch) {
  constexpr int64_t kBlocks = int64_t(0xFFFFFFFF) / C::block;
  for (int64_t b = 0; b < blocks; b += kBlocks)
    launch(dim3((unsigned)(blocks - b < kBlocks ? blocks - b : kBlocks)), b);
  return hipGetLastError();
}

template <class C>
hipError_t launch_reduce(const int32_t* in, int64_t n, const int64_t* offsets, int64_t S,
                         int64_t* out, void* ws, hipStream_t s, bool persistent) {
  const SegWs w = carve(ws, n, S, false);
  const int64_t units = S + (n + C::unit - 1) / C::unit;   // at least the units of the call
  const bool many_short = short_reduce(n, S, persistent);
  if (persistent && !many_short) {
    static int resident[64] = {0};
    int64_t g = launch::resident_grid(seg_reduce_persistent_kernel<C>, resident, 1, C::block);
    if (g > units) g = units;
    if (g > kMaxReduceBlocks) g = kMaxReduceBlocks;
    hipLaunchKernelGGL(seg_reduce_persistent_kernel<C>, dim3((unsigned)g), dim3(C::block), 0, s,
                       in, n, offsets, S, out, w.words, (WsHeader*)ws);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((plan_kernel<C, false>), dim3(1), dim3(kPlanBlock), 0, s, offsets, n, S,
                     w.total, w.unit_start, out, (uint64_t*)nullptr, (int64_t)0);
  if (many_short)
    return in_grids<C>((units + C::waves - 1) / C::waves, [&](dim3 grid, int64_t block0) {
      hipLaunchKernelGGL(seg_reduce_short_kernel<C>, grid, dim3(C::block), 0, s, in, n, offsets, S,
                         w.total, units, w.unit_start, out, block0);
    });
  return in_grids<C>(units, [&](dim3 grid, int64_t block0) {
    hipLaunchKernelGGL(seg_reduce_kernel<C>, grid, dim3(C::block), 0, s, in, n, offsets, S, w.total,
                       w.unit_start, out, block0);
  });
}

// The scan stays in the two-launch form: in a persistent grid the units of
// one round run together, so a unit's look-back finds its predecessors still
// running, where in-order dispatch has started them earlier (measured on the
// 4096-segment workload: 535 us against 469 us).
template <class C>
hipError_t launch_scan(const int32_t* in, int32_t* out, int64_t n, const int64_t* offsets,
                       int64_t S, void* ws, hipStream_t s) {
  const SegWs w = carve(ws, n, S, true);
  const int64_t mu = S + (n + C::unit - 1) / C::unit;
  hipLaunchKernelGGL((plan_kernel<C, true>), dim3(1), dim3(kPlanBlock), 0, s, offsets, n, S,
                     w.total, w.unit_start, (int64_t*)nullptr, w.status, mu);
  if (short_scan(n, S))
    return in_grids<C>((mu + C::waves - 1) / C::waves, [&](dim3 grid, int64_t block0) {
      hipLaunchKernelGGL(seg_scan_short_kernel<C>, grid, dim3(C::block), 0, s, in, out, n, offsets,
                         S, w.total, mu, w.unit_start, w.status, (WsHeader*)ws, block0);
    });
  return in_grids<C>(mu, [&](dim3 grid, int64_t block0) {
    hipLaunchKernelGGL(seg_scan_kernel<C>, grid, dim3(C::block), 0, s, in, out, n, offsets, S,
                       w.total, w.unit_start, w.status, (WsHeader*)ws, block0);
  });
}

// The reduce has no 64K unit: holding 16 rounds in 1024 threads spills.
constexpr const char* kReduceNames[] = {"unit8k", "unit16k", "unit32k", "unit32k_w16", "by_mean"};
constexpr const char* kScanNames[] = {"unit8k",      "unit16k",     "unit32k",
                                      "unit32k_w16", "unit64k_w16", "by_mean"};
constexpr int kReduceByMean = 4, kScanByMean = 5;
constexpr int kReduceDefaults[tune::kClasses] = {kReduceByMean, kReduceByMean, kReduceByMean,
                                                 kReduceByMean};
constexpr int kScanDefaults[tune::kClasses] = {kScanByMean, kScanByMean, kScanByMean, kScanByMean};
const bool kRegistered =
    (tune::register_op(tune::kSegReduceI32, "seg_reduce_i32", 5, kReduceNames, kReduceDefaults),
     tune::register_op(tune::kSegScanI32, "seg_scan_i32", 6, kScanNames, kScanDefaults), true);

}  // namespace

namespace launch {

size_t segmented_workspace(int64_t n, int64_t S, bool scan) {
  return (size_t)(sizeof(WsHeader) + 64 + round64(state_words(n, S, scan) * 8) + (S + 1) * 8);
}

int64_t segmented_max_grid(int64_t n, int64_t S) { return max_units(n, S); }

hipError_t reduce_segmented_i32(const int32_t* in, int64_t n, const int64_t* offsets, int64_t S,
                                int64_t* out, void* ws, hipStream_t s, bool persistent) {
  (void)kRegistered;
  int c = tune::get(tune::kSegReduceI32, tune::size_class(tune::kSegReduceI32, n));
  persistent = persistent && persistent_fits(n, S);
  if (c == kReduceByMean) c = reduce_by_mean(n, S, persistent);
  switch (c) {
    case 1: return launch_reduce<UnitCfg<256, 16>>(in, n, offsets, S, out, ws, s, persistent);
    case 2: return launch_reduce<UnitCfg<512, 16>>(in, n, offsets, S, out, ws, s, persistent);
    case 3: return launch_reduce<UnitCfg<1024, 8>>(in, n, offsets, S, out, ws, s, persistent);
    default: return launch_reduce<UnitCfg<256, 8>>(in, n, offsets, S, out, ws, s, persistent);
  }
}

hipError_t scan_segmented_i32(const int32_t* in, int32_t* out, int64_t n, const int64_t* offsets,
                              int64_t S, void* ws, hipStream_t s) {
  (void)kRegistered;
  int c = tune::get(tune::kSegScanI32, tune::size_class(tune::kSegScanI32, n));
  if (c == kScanByMean) c = scan_by_mean(n, S);
  switch (c) {
    case 1: return launch_scan<UnitCfg<256, 16>>(in, out, n, offsets, S, ws, s);
    case 2: return launch_scan<UnitCfg<512, 16>>(in, out, n, offsets, S, ws, s);
    case 3: return launch_scan<UnitCfg<1024, 8>>(in, out, n, offsets, S, ws, s);
    case 4: return launch_scan<UnitCfg<1024, 16>>(in, out, n, offsets, S, ws, s);
    default: return launch_scan<UnitCfg<256, 8>>(in, out, n, offsets, S, ws, s);
  }
}

}  // namespace launch
}  // namespace desc
