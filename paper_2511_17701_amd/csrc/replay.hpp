// replay.hpp -- the iterates of a fixed-point iteration, last to first.
#pragma once

#include <hip/hip_runtime.h>

namespace grpic {

// Calls visit(y1, y2) with the iterates n - 1, ..., 0 of y <- step(y) from (y1,
// y2), iterate 0.  On the way forward the first iterate of each of up to kKeep
// segments is kept; backwards each segment's iterates are computed again from
// it, kKeep of them at a time (segments are longer than that for n > kKeep^2,
// and are then walked again for each kKeep).
template <int kKeep, class Step, class Visit>
__host__ __device__ inline void reverse_iterates(int n, double y1, double y2, Step step, Visit visit) {
  double keep[kKeep][2], seg[kKeep][2];
  const int len = (n + kKeep - 1) / kKeep;  // iterates per segment
  for (int it = 0; it < n; ++it) {
    if (it % len == 0) {
      keep[it / len][0] = y1;
      keep[it / len][1] = y2;
    }
    step(y1, y2);
  }
  int have = n;  // seg holds the iterates [have, have + kKeep)
  for (int it = n - 1; it >= 0; --it) {
    if (it < have) {
      const int first = it / len * len;
      have = first > it - (kKeep - 1) ? first : it - (kKeep - 1);
      y1 = keep[it / len][0];
      y2 = keep[it / len][1];
      for (int q = first; q <= it; ++q) {
        if (q >= have) {
          seg[q - have][0] = y1;
          seg[q - have][1] = y2;
        }
        step(y1, y2);
      }
    }
    visit(seg[it - have][0], seg[it - have][1]);
  }
}

}  // namespace grpic
