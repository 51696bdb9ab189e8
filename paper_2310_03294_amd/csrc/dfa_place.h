// How long workgroups of two kinds take, placed as the hardware does it: in order, one per CU, each XCD its range of
// them (XcdMap).  For the estimates by which a call's work is divided.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

namespace dfa {

constexpr int XCDS = 8, CUS = 32;      // CUs of an XCD

// Workgroups of one kind on an XCD: how many, us of the longest and in the mean, tiles of a head.
struct Kind { int64_t n; double longest, mean; int64_t per_head; };

// When na workgroups of `a` us and then nb of `b` are done on an XCD.
inline double placed(int64_t na, double a, int64_t nb, double b) {
  const int64_t late = na % CUS, early = CUS - late;                 // CUs that are free at t2, at t1
  const double t1 = static_cast<double>(na / CUS) * a, t2 = late ? t1 + a : t1;
  if (!nb) return t2;
  double least = t1 + nb * b / early;
  if (least > t2) least = (nb * b + early * t1 + late * t2) / CUS;
  double end = 1e30;
  for (double t0 : {t1, t2}) {         // a workgroup of the second kind ends last, on a CU of either sort
    double n = std::max(1., std::ceil((least - t0) / b - 1e-9));
    for (int k = 0; k < 3; ++k, ++n) {
      const double t = t0 + n * b;
      const int64_t done = early * static_cast<int64_t>((t - t1) / b + 1e-9) + (t > t2 ? late * static_cast<int64_t>((t - t2) / b + 1e-9) : 0);
      if (done >= nb) { end = std::min(end, t); break; }
    }
  }
  return std::max(t2, end);
}

// Workgroups of kind a and then b.  Of a causal call they are of all lengths, a head's longest first: the even share and `tail` of the
// shorter kind's longest, but the last head's longest workgroup may begin late (`late` of a mean workgroup before the even share of
// what comes before it, after the shortest one at least).
inline double makespan(const Kind& a, const Kind& b, bool causal, double shortest, double tail, double late) {
  if (!causal) return placed(a.n, a.longest, b.n, b.longest);
  const double alone = std::max(a.n ? a.longest : 0., b.n ? b.longest : 0.);
  if (a.n + b.n <= CUS) return alone;
  const int64_t before = std::max<int64_t>(0, b.n - b.per_head);      // of the second kind, before the last head's
  const double share = (a.n * a.mean + b.n * b.mean) / CUS;
  const double begin = a.n + before < CUS ? 0. : std::max(shortest, (a.n * a.mean + before * b.mean) / CUS - late * (before < CUS ? a : b).mean);
  return std::max(alone, std::max(begin + (b.n ? b.longest : 0.), share + tail * std::min(a.longest, b.longest)));
}

// A causal call's (head, part) groups go to the XCDs in ranges, longest tiles first: with a part of a group left over, an XCD that
// gets its first tiles has so much more than an even share.
inline double uneven(int64_t groups) {
  const double g = static_cast<double>(groups) / XCDS, whole = static_cast<double>(groups / XCDS), rest = g - whole;
  return groups <= 2 ? 1.0 : (whole + rest * (2 - rest)) / g;
}

}  // namespace dfa
