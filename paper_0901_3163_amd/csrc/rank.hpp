// Ranks of the eigenvalue keys of the projected problems.  The ranks are used as indices, so the order
// has to be total whatever the keys hold: a comparison by < and == alone gives every NaN rank 0,
// and then some ranks belong to nobody.  NaN comes after every number here and ties go by index, so
// that n keys always have n different ranks and a NaN travels on in the data, to the host's check.
#pragma once

#include <cmath>

#if defined(__HIPCC__)
#define DL_HD __host__ __device__
#else
#define DL_HD
#endif

namespace dl {

// Key a of index i comes before key b of index j.
DL_HD inline bool key_before(double a, int i, double b, int j) {
  const bool an = a != a, bn = b != b;
  if (an || bn) return an == bn ? i < j : bn;
  return a < b || (a == b && i < j);
}

// The same by magnitude, then value, then index.
DL_HD inline bool key_before_abs(double a, int i, double b, int j) {
  const double x = std::fabs(a), y = std::fabs(b);
  return x < y || (!(y < x) && key_before(a, i, b, j));
}

// Keys that come before key i.
DL_HD inline int key_rank(int n, const double* key, int i) {
  int r = 0;
  for (int j = 0; j < n; ++j) r += key_before(key[j], j, key[i], i);
  return r;
}
DL_HD inline int key_rank_abs(int n, const double* key, int i) {
  int r = 0;
  for (int j = 0; j < n; ++j) r += key_before_abs(key[j], j, key[i], i);
  return r;
}

}  // namespace dl
