// The search direction of a refinement sweep (api.hip, pcg.hip): plain C++.
#pragma once

namespace bfal {

// out = z + sum a_j p_j (FP64), the terms added in their order.
//
// The directions kept are a ring of kMax buffers and the new one takes the
// oldest one's, so the oldest direction is not there any more when its term's
// turn comes: the term finds the sum so far in its place and scales it by
// 1 + a.  The step along the direction is an exact line search, so the scale
// does not change it; the new direction is conjugate to the other kMax - 1.
// Only a = -1 must not be taken: nothing would be left of the direction, and
// the sweep would end as if the matrix were not positive definite.
struct Directions {
  static constexpr int kMax = 4;
  int n = 0;
  double a[kMax];
  const double* p[kMax];

  void add(double aj, const double* pj, const double* out) {
    if (pj == out && aj == -1.0) return;
    a[n] = aj;
    p[n++] = pj;
  }
};

}  // namespace bfal
