// Tau-steps that the accelerated RKL iteration (App. A.4) needs on a coarsest
// level for given tolerances: the rule by which a plan's V-cycles may solve that
// level directly instead.  Host arithmetic only.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <vector>

namespace rkl {

struct AccelSteps {
  int loose, tight;  // 0: not within 200 steps
};

// The steps (at most 200) after which the schedule `sched` has reduced every
// residual on a level of ns[d] cells of spacing hs[d] to `loose` and to `tight`
// (loose >= tight) of its right-hand side: the largest product of the steps'
// stage polynomials P_s over the spectrum, sampled at 2048 evenly and 512
// logarithmically spaced |lambda| and at its ends.  (Between the samples of a
// polynomial with more lobes than that a product may be a little larger.)
//
// The schedule's stage counts grow and its last one repeats, so the recursion
// P_j runs once, up to the largest count, for all samples together with its
// coefficients outside their loop, and both tolerances are read off the same
// products.  A plan's creation waits for it: 50 x 30 x 22 cells 7.7 -> 0.2 ms, 250^3
// 74 -> 0.5, a spacing ratio that takes 4096 stages 1380 -> 6 from one recursion
// per step, sample and tolerance.
inline AccelSteps accel_steps(const int ns[3], const double hs[3], double dtpar, bool periodic, double theta,
                              const std::vector<int>& sched, double loose, double tight) {
  double lo = periodic ? HUGE_VAL : 0.0, hi = 0.0;
  for (int d = 0; d < 3; ++d) {
    if (ns[d] == 1 && (periodic || std::isinf(hs[d]))) continue;
    const double w = 4.0 / (hs[d] * hs[d]);
    if (periodic) {
      lo = std::min(lo, w * std::pow(std::sin(M_PI / ns[d]), 2));
      hi += w * std::pow(std::sin(M_PI * (ns[d] / 2) / ns[d]), 2);
    } else {
      lo += w * std::pow(std::sin(M_PI / (2.0 * ns[d])), 2);
      hi += w;
    }
  }
  AccelSteps out{0, 0};
  if (!(lo > 0.0) || !(hi >= lo) || !std::isfinite(hi) || sched.empty()) return out;
  std::vector<double> x;
  for (int q = 0; q <= 2048; ++q) x.push_back(lo + (hi - lo) * q / 2048.0);
  for (int q = 1; q < 512; ++q) x.push_back(lo * std::pow(hi / lo, q / 512.0));
  for (double& v : x) v = 1.0 - theta * dtpar * v;
  const size_t n = x.size();
  // p1 = P_j and p0 = P_{j-1} at the samples
  std::vector<double> p0(n, 1.0), p1(x), amp(n, 1.0);
  int j = 1;
  for (int step = 0; step < 200; ++step) {
    const int s = sched[std::min<size_t>(step, sched.size() - 1)];
    if (s < j) {
      std::fill(p0.begin(), p0.end(), 1.0);
      p1 = x;
      j = 1;
    }
    for (; j < s;) {
      ++j;
      const double a = (2.0 * j - 1.0) / j, b = (j - 1.0) / j;
      for (size_t q = 0; q < n; ++q) {  // P_j = a x P_{j-1} - b P_{j-2}
        const double pn = a * x[q] * p1[q] - b * p0[q];
        p0[q] = p1[q];
        p1[q] = pn;
      }
    }
    double worst = 0.0;
    for (size_t q = 0; q < n; ++q) {
      amp[q] *= p1[q];
      worst = std::max(worst, std::fabs(amp[q]));
    }
    if (out.loose == 0 && worst <= loose) out.loose = step + 1;
    if (worst <= tight) {
      out.tight = step + 1;
      return out;
    }
    if (!(worst < 1e6)) return out;
  }
  return out;
}

}  // namespace rkl
