// Output rows per segment of a first layer's strips (stem.hip).  Host arithmetic only: no HIP header is needed to compile this file.
#pragma once

namespace octo {

// A strip walked by one wavefront is a serial chain (11 crops of 224 x 224 have 22 strips of 112 rows, the chip has 2048 wavefronts).  Cut
// into segments it costs, with the pool, one more convolution row for each cut, and about two rows' time to start; the length with the
// shortest busiest wavefront is taken.  Only the shortest length for each number of segments is looked at, some 2 sqrt(out_h) of them, since
// the answer is worked out for every launch: 640 rows one by one took the host 3.7 us, these 0.6.
inline int stem_segment(int out_h, long long strips, long long waves, bool pool) {
  long long best = 0;
  int pick = 1;
  for (int seg = out_h; seg >= 1; --seg) {
    const int cuts = (out_h + seg - 1) / seg;
    seg = (out_h + cuts - 1) / cuts;
    const long long rounds = (strips * cuts + waves - 1) / waves, rows = rounds * (pool ? 2 * seg + 3 : seg + 2);
    if (seg == out_h || rows < best) { best = rows; pick = seg; }
  }
  return pick;
}

}  // namespace octo
