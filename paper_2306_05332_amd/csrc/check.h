// The convergence test of a cycle, by one workgroup: shared by its own kernel
// (kernels.hip) and by the coarse tail, which runs it for small grids
// (tail_col.hip).
//
// rel = sqrt(sum of part[b * stride]) / sqrt(res0sq) for the state at the start
// of cycle cs->m; records it and decides, in this order:
// non-finite -> RKL_ENONFINITE; rel <= tol -> done; three consecutive
// increases that end above twice the best residual so far -> RKL_EDIVERGED;
// with tol > 0, the last eight states all above 0.9 of the best state
// before them (the residual has stopped falling, as it does at the float64
// rounding floor of M u - f, about eps Lambda ||u|| / ||f||) -> RKL_ENOCONV,
// marked stalled (tol = 0 asks for exactly max_cycles cycles);
// m >= max_cycles -> RKL_ENOCONV.  Also stores the mean of the residual
// (part[b * stride + 1] / count) as a diagnostic.
//
// A few kilobytes are read once a cycle, so it is latency only: everything is
// requested by check_load before anything is waited for, and the history's
// minima are taken by one wavefront's lanes, only where a decision needs them (one
// thread walking the history after two block sums: 5.7 us at 256^3, now 4.6).
#pragma once

#include "kernels.h"

namespace rkl {

struct CheckLoads {
  double v2, v1;       // the thread's share of the sums
  double r0, h;        // res0^2; wavefront 0: history entry of the lane
  double last0, last1, last2, last3;
  int m;
};

// nt: threads of the workgroup
__device__ __forceinline__ void check_load(const CheckArgs& A, int nt, CheckLoads& L) {
  L.v2 = L.v1 = 0.0;
  for (int b = threadIdx.x; b < A.nblk; b += nt) {
    L.v2 += A.part[(size_t)b * A.stride];
    if (A.stride > 1) L.v1 += A.part[(size_t)b * A.stride + 1];
  }
  L.m = A.cs->m;
  L.r0 = A.res0sq[0];
  L.h = L.last0 = L.last1 = L.last2 = L.last3 = HUGE_VAL;
  if (threadIdx.x < WAVE) {
    L.h = A.cs->hist[threadIdx.x];
    L.last0 = A.cs->last[0];
    L.last1 = A.cs->last[1];
    L.last2 = A.cs->last[2];
    L.last3 = A.cs->last[3];
  }
}

// sh: 2 NT / 64 doubles that no thread still reads; every thread calls it
template <int NT>
__device__ __forceinline__ void check_finish(const CheckArgs& A, const CheckLoads& L, double* sh) {
  const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
  constexpr int NW = NT / WAVE;
  static_assert(NW <= WAVE, "one lane per wavefront");
  const double p2 = wave_sum_dpp(L.v2), p1 = wave_sum_dpp(L.v1);
  if (lane == 0) {
    sh[w] = p2;
    sh[NW + w] = p1;
  }
  __syncthreads();
  if (w != 0) return;
  ConvState* cs = A.cs;
  const double t2 = wave_sum_dpp(lane < NW ? sh[lane] : 0.0);
  const double t1 = wave_sum_dpp(lane < NW ? sh[NW + lane] : 0.0);
  const double rel = sqrt(t2) / sqrt(L.r0);
  const int m = L.m;
  const int hmax = m < CONV_HIST ? m : CONV_HIST;
  // states m - 1, m - 2, m - 3
  auto last = [&](int q) {
    const double lo = q & 1 ? L.last1 : L.last0, hi = q & 1 ? L.last3 : L.last2;
    return q & 2 ? hi : lo;
  };
  const double l1 = last(m + 3), l2 = last(m + 2), l3 = last(m + 1);
  constexpr int SW = 8;  // stall window
  // best of the history's states q <= hi (or, without `below`, q > hi)
  auto best = [&](int hi, bool below) {
    double v = HUGE_VAL;
    for (int q = lane; q < hmax; q += WAVE)
      if ((q <= hi) == below) v = fmin(v, q < WAVE ? L.h : cs->hist[q]);
#pragma unroll
    for (int off = WAVE / 2; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off, WAVE));
    return v;
  };
  int status = 1;  // 1: keep going
  int stalled = 0;
  if (!isfinite(rel)) status = -5;
  else if (rel <= A.tol) status = 0;
  else if (m >= 3 && rel > l1 && l1 > l2 && l2 > l3 && rel > 2.0 * best(m - 3, true)) status = -4;
  else if (A.tol > 0.0 && m >= SW && m < CONV_HIST && fmin(rel, best(m - SW, false)) > 0.9 * best(m - SW, true)) {
    status = -3;
    stalled = 1;
  } else if (m >= A.max_cycles) status = -3;
  if (lane != 0) return;
  cs->mean = t1 / A.count;
  if (m < CONV_HIST) cs->hist[m] = rel;
  cs->last[m & 3] = rel;
  cs->rel = rel;
  if (status != 1) {
    cs->status = status;
    cs->stalled = stalled;
    cs->result_m = m;
    cs->stop = 1;
  } else {
    cs->m = m + 1;
  }
}

}  // namespace rkl
