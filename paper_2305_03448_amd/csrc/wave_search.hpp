// wave_search.hpp -- search of a nondecreasing array by one whole wave: which
// problem (grouped.hip) or segment (segmented.hip) a global index belongs to.
#pragma once
#include "common.hpp"
#include "layouts.hpp"
#include "view.hpp"

namespace desc {

// Last i in [0, G) with start[i] <= t, for a nondecreasing start with
// start[0] <= t < start[G]: a 64-way search by one whole wave.  Each round
// every lane reads one boundary and a ballot counts those <= t (a prefix of
// the lanes), so G = 512 takes two rounds of parallel loads instead of nine
// dependent ones.
template <class T>
__device__ __forceinline__ idx_t wave_owner(const T* start, int64_t G, int64_t t) {
  auto st = array(start, G);
  const idx_t lane = lane_of_wave().index();
  layout::Search64 s{0, G};
  while (!s.done()) {
    const idx_t i = s.entry(lane);
    s = s.next(__popcll(__ballot(i < s.hi && st[i] <= t)));
  }
  return s.lo;
}

}  // namespace desc
