// Decay of the inverse of T = 1 + i tau H (real potential, off-diagonals of magnitude kappa), on the
// host: which joints decouple and how far a cut of the line is felt.  The rules that choose one-pass
// forms, levels and halos rest on these alone.
//
// Conjugating T by exp(eta j) changes its Hermitian part, the identity, by at most
// theta = 2 kappa sinh(eta), whatever the potential is; so for theta < 1
//     |(T^-1)_ij| <= exp(-eta |i - j|) / (1 - theta),
// and a step's conjugated norm is at most (1 + theta) / (1 - theta) (Combes and Thomas's argument).
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>

// Minimum of f over eta in (0, hi) by golden-section search (f has one minimum there).
template <typename F>
double min_over(double hi, const F& f) {
  const double g = 0.6180339887498949;
  double a = 0.0, b = hi, x1 = b - g * (b - a), x2 = a + g * (b - a), f1 = f(x1), f2 = f(x2);
  for (int i = 0; i < 48; ++i) {
    if (f1 < f2) {
      b = x2;
      x2 = x1;
      f2 = f1;
      x1 = b - g * (b - a);
      f1 = f(x1);
    } else {
      a = x1;
      x1 = x2;
      f1 = f2;
      x2 = a + g * (b - a);
      f2 = f(x2);
    }
  }
  return std::min(f1, f2);
}
inline double eta_max(double kap) { return kap > 0.0 ? std::min(8.0, std::asinh(0.5 / kap)) : 8.0; }

// Whether two joint lines B rows apart are decoupled to 2^-66 in every real potential: their
// coupling kappa^2 (T^-1)_{1,m} against a diagonal of real part at least 1.
inline bool decoupled(double kap, double B) {
  return min_over(eta_max(kap), [&](double e) {
    const double th = std::min(2.0 * kap * std::sinh(e), 1.0 - 1e-12);
    return 2.0 * std::log(std::max(kap, 1e-30)) - e * (B - 2.0) - std::log(1.0 - th);
  }) <= -66.0 * M_LN2;
}

// Rows that a cut of the line has to stay away after s steps (nshaped_windows.hpp): the smallest
// D with r^s exp(-eta D) / (2 sinh eta) <= 2^-70 for some eta.
inline double window_halo(double kap, int64_t s) {
  return std::ceil(min_over(eta_max(kap), [&](double e) {
    const double th = std::min(2.0 * kap * std::sinh(e), 1.0 - 1e-12);
    return (70.0 * M_LN2 + (double)s * std::log((1.0 + th) / (1.0 - th)) -
            std::log(2.0 * std::sinh(e))) / e;
  })) + 1.0;
}

// Levels of lane blocks of M rows whose reduced systems are diagonal (joints M * 2^levels rows
// apart), the least of `count` from `least` on, or -1.
inline int decay_levels(double kap, int M, int least, int count) {
  for (int lv = least; lv < least + count; ++lv)
    if (decoupled(kap, (double)(M << lv))) return lv;
  return -1;
}
