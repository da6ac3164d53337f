// eigorder.h -- the order of eigenvalues that the projected eigensolvers return.
#pragma once

namespace adc2 {

// Whether eigenvalue u at place j comes before eigenvalue v at place i: ascending,
// equal ones by place, NaN after every number.  A total order, so that counting the
// places before each one gives a permutation whatever the values.  (constexpr: host
// and device.)
constexpr bool eig_before(double u, int j, double v, int i) {
  const bool un = u != u, vn = v != v;
  if (un || vn) return vn && (!un || j < i);
  return u < v || (u == v && j < i);
}

}  // namespace adc2
