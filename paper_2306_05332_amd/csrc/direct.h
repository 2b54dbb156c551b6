// Direct coarsest solve: device building block shared by the one-workgroup
// coarse tail (tail.hip) and the multi-workgroup form (direct.hip).
//
// The coarsest operator has constant coefficients on a box, so it is a sum of
// three one-dimensional operators with known orthonormal eigenvectors: sines
// sqrt(2/n) sin(pi (k+1)(i+1/2)/n) for the homogeneous ghost -u, cosines and
// sines of 2 pi k i / n for a periodic axis.  With Q_d the matrix whose rows
// are axis d's eigenvectors, M u = b is solved by
//   u = (Qx x Qy x Qz)^T [ (Qx x Qy x Qz) b / lambda ],
// six applications of a small dense matrix along one axis.  Each is a
// contraction, done in 16 x 16 x 4 float64 matrix instructions whatever the
// precision of the level.
#pragma once

#include "kernels.h"

namespace rkl {

typedef double dbl4 __attribute__((ext_vector_type(4)));

// One matrix application along an axis of n cells and element stride s, by the
// wavefronts w, w + nw, ... of a workgroup: lines q = 0 .. nlines - 1 of the
// axis start at element (q / s) (n s) + q % s of `in` and `out` (distinct
// arrays).  out[k] = sum_j Q[k][j] in[j], or with INV out[j] = sum_k Q[k][j]
// in[k].  A tile is 16 lines by 16 rows of the result.  Lane layout of the
// instruction: A row l & 15, column l >> 4; B row l >> 4, column l & 15;
// result rows 4 v + (l >> 4), column l & 15.  `sc` (the result's row, its
// line, its value) gives the value stored.
template <bool INV, typename F>
__device__ __forceinline__ void axis_apply(const double* in, double* out, const double* Q, int n, int s, int nlines,
                                           int w, int nw, int lane, F&& sc) {
  const int ntm = (n + 15) >> 4, ntl = (nlines + 15) >> 4;
  const int r = lane & 15, kq = lane >> 4;
  for (int t = w; t < ntm * ntl; t += nw) {
    const int m0 = (t % ntm) << 4, q = ((t / ntm) << 4) + r;
    const bool lok = q < nlines;
    const int base = lok ? (q / s) * (n * s) + q % s : 0;
    const int i = m0 + r;
    dbl4 acc = {0.0, 0.0, 0.0, 0.0};
    // four steps' operands are loaded before the first is used (a step at a time,
    // the latencies of the matrix loads added up: planes of 50 x 30 took 13.4 and
    // 11.7 us forth and back in four wavefronts, 6.9 and 6.3 now in eight);
    // out-of-range entries read the last one in range and count as 0
    const int ic = min(i, n - 1);
    for (int k0 = 0; k0 < n; k0 += 16) {
      double a[4], b[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = min(k0 + 4 * u + kq, n - 1);
        a[u] = INV ? Q[k * n + ic] : Q[ic * n + k];
        b[u] = in[base + k * s];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool kok = k0 + 4 * u + kq < n;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(i < n && kok ? a[u] : 0.0, lok && kok ? b[u] : 0.0, acc, 0, 0, 0);
      }
    }
    if (lok) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int k = m0 + 4 * v + kq;
        if (k < n) out[base + k * s] = sc(k, q, acc[v]);
      }
    }
  }
}

}  // namespace rkl
