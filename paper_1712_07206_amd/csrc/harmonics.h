// Real and complex harmonics: the unitary map between them at fixed l, and row indices.
#pragma once

#include <hip/hip_runtime.h>

namespace hsb {

// c(l,m,mu): the coefficient of s_{l,mu} in i^l conj(Y_lm); nonzero for |m| = |mu| only.  Without
// its factor 1/sqrt(2) (m != 0) it is a power of i times a sign: power e of i.
__device__ inline int harmonic_power(int l, int m, int mu) {
  // m > 0: c = i^l (s_m - i s_-m);  m < 0: c = (-1)^m i^l (s_|m| + i s_-|m|)
  int e = l;
  if (m < 0 && (m & 1)) e += 2;
  if (mu < 0) e += m > 0 ? 3 : 1;
  return e & 3;
}

__device__ inline double2 times_i(double2 v, int e) {
  switch (e & 3) {
    case 0: return v;
    case 1: return make_double2(-v.y, v.x);
    case 2: return make_double2(-v.x, -v.y);
    default: return make_double2(v.y, -v.x);
  }
}

__device__ inline void lm_of(int L, int& l, int& m) {
  l = (int)sqrt((double)L + 0.5);
  m = L - l * l - l;
}

}  // namespace hsb
