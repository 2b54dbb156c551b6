// Two-dimensional levels of the V-cycle, one launch per stroke.
//
// The strokes of brick.hip on a two-dimensional level (eq. discrete_laplace_2D):
//   down  all n_pre tau-steps (Sec. 2.1 step 1; App. A), the residual and its
//         restriction (steps 2a-2b, the 4-child average),
//   up    prolongation and correction (steps 4-5, bilinear), then the n_post
//         tau-steps.
// A workgroup takes a window of 64 columns by SEG segments of LEN rows, halo
// included; a wavefront owns one segment, a lane one column of it in registers.
// x neighbours come by wavefront shifts, y neighbours are the lane's own cells,
// and only a segment's first and last row go through LDS, so a stage costs two
// LDS writes, two reads and a barrier for LEN cells.  A level is read and written
// once per stroke: u, b and the output, where the pair of tau-steps, the
// residual + restriction, the prolongation and the tau-step took four passes.
// Values outside the exact region grow stale by one cell a stage and are never
// written; ghosts as in Sec. 2.3.
//
// Measured, float64 periodic, separate passes -> here: 4096^2 down 129 -> 105 us
// (4.2 TB/s of compulsory traffic), up 108 -> 85 (5.1 TB/s; both bound by memory);
// 2048^2 36 -> 20.4 and 31 -> 20.6; 512^2 13 -> 5.2 and 14 -> 5.2 (bound by the
// chain of one burst, a barrier a stage and one store).  4096^2 solve 4.45 -> 3.39
// ms, 256^2 cycle 89 -> 61 us.
#include "host_common.h"
#include "kernels.h"

namespace rkl {

constexpr int W2S = 4;  // most stages per stroke

template <typename T>
struct W2Args {
  int nx, ny;
  int tx, nblk;        // tiles in x, all tiles
  int hx, hy, ox, oy;  // halo and exact cells of a window
  int s, stages;       // stages per tau-step and in all
  T ihx, ihy;
  T co[W2S][3];        // mu, nu, c of a tau-step's stages (mu_1 = 1, nu_1 = 0)
};

template <typename T, bool PER, int LEN, int SEG>
struct Win2 {
  int i, k0;    // lane's column and the segment's first row in the window
  int gx, gy;   // and in the level (unwrapped)
  int cx, y0;   // wrapped column and first row
  bool gxm, gxp, xin;
  int zlo, zhi;  // cells next to the y faces (Dirichlet; else -1)
  int sm, sp;    // segments below and above (the segment itself at the window's ends)

  __device__ __forceinline__ Win2(const W2Args<T>& A, int tile) {
    i = threadIdx.x & 63;
    const int seg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    k0 = seg * LEN;
    gx = (tile % A.tx) * A.ox - A.hx + i;
    gy = (tile / A.tx) * A.oy - A.hy + k0;
    gxm = !PER && gx == 0;
    gxp = !PER && gx == A.nx - 1;
    zlo = PER ? -1 : -gy;
    zhi = PER ? -1 : A.ny - 1 - gy;
    xin = PER || (gx >= 0 && gx < A.nx);
    cx = PER ? ((gx % A.nx) + A.nx) % A.nx : gx;
    y0 = PER ? ((gy % A.ny) + A.ny) % A.ny : gy;
    sm = seg > 0 ? seg - 1 : seg;
    sp = seg < SEG - 1 ? seg + 1 : seg;
  }
  __device__ __forceinline__ int seg() const { return k0 / LEN; }
  // the lane's cells of a level array (0 outside a Dirichlet box)
  __device__ __forceinline__ void load(const W2Args<T>& A, const T* __restrict__ g, T (&v)[LEN]) const {
    int y = y0;
#pragma unroll
    for (int m = 0; m < LEN; ++m) {
      v[m] = (T)0;
      if (xin && (PER || (y >= 0 && y < A.ny))) v[m] = (g + (size_t)y * A.nx)[cx];
      ++y;
      if (PER && y == A.ny) y = 0;
    }
  }
  __device__ __forceinline__ bool xown(const W2Args<T>& A) const {
    return i >= A.hx && i < A.hx + A.ox && gx < A.nx;
  }
  // row m is one of the window's exact rows, in the box (uniform)
  __device__ __forceinline__ bool yown(const W2Args<T>& A, int m) const {
    return k0 + m >= A.hy && k0 + m < A.hy + A.oy && gy + m < A.ny;
  }
  __device__ __forceinline__ void store(const W2Args<T>& A, T* __restrict__ g, const T (&v)[LEN]) const {
    const bool xo = xown(A);
#pragma unroll
    for (int m = 0; m < LEN; ++m)  // exact cells are never wrapped
      if (yown(A, m) && xo) (g + (size_t)(gy + m) * A.nx)[gx] = v[m];
  }
  // the segment's end rows into E[seg][2][64]
  __device__ __forceinline__ void put(T* E, const T (&v)[LEN]) const {
    E[seg() * 128 + i] = v[0];
    E[seg() * 128 + 64 + i] = v[LEN - 1];
  }
  // M y at the lane's cells, E holding the end rows of every segment
  __device__ __forceinline__ void lap(const W2Args<T>& A, const T* E, const T (&y)[LEN], T (&out)[LEN]) const {
    const T zl = E[sm * 128 + 64 + i], zh = E[sp * 128 + i];
#pragma unroll
    for (int m = 0; m < LEN; ++m) {
      const T c = y[m];
      T xm = wshift<DPP_WAVE_SHR1>(c), xp = wshift<DPP_WAVE_SHL1>(c);
      T zm = m > 0 ? y[m > 0 ? m - 1 : 0] : zl;
      T zp = m + 1 < LEN ? y[m + 1 < LEN ? m + 1 : m] : zh;
      if (!PER) {
        if (gxm) xm = -c;
        if (gxp) xp = -c;
        if (m == zlo) zm = -c;
        if (m == zhi) zp = -c;
      }
      out[m] = fma_of((zm + zp) - (T)2 * c, A.ihy, ((xm + xp) - (T)2 * c) * A.ihx);
    }
  }
  // the stroke's stages from y, whose end rows `cur` holds too unless ZERO (the
  // zero iterate, whose first stage is pointwise); with LAST the result's end
  // rows are left in `cur` (after a barrier).  r2: sum of (M y - b)^2 of the
  // starting y over the lane's exact cells.
  template <bool ZERO, bool LAST, bool SUM>
  __device__ __forceinline__ void relax(const W2Args<T>& A, T*& cur, T*& alt, T (&y)[LEN], const T (&b)[LEN],
                                        double& r2) const {
    T y2[LEN];
    int q = 0;
    for (int t = 0; t < A.stages; ++t) {
      const T mu = A.co[q][0], nu = A.co[q][1], c = A.co[q][2];
      T w[LEN];
      if (ZERO && t == 0) {
#pragma unroll
        for (int m = 0; m < LEN; ++m) w[m] = (T)0;
      } else {
        lap(A, cur, y, w);
      }
      if (q == 0) {
        const bool xo = SUM && t == 0 && xown(A);
#pragma unroll
        for (int m = 0; m < LEN; ++m) {
          const T res = w[m] - b[m];
          if (SUM && xo && yown(A, m)) r2 += (double)res * (double)res;
          y2[m] = y[m];
          y[m] = fma_of(c, res, y[m]);
        }
      } else {
#pragma unroll
        for (int m = 0; m < LEN; ++m) {
          const T res = w[m] - b[m];
          const T v = rkl_stage(mu, y[m], nu, y2[m], c, res);
          y2[m] = y[m];
          y[m] = v;
        }
      }
      q = q + 1 == A.s ? 0 : q + 1;
      if (LAST || t + 1 < A.stages) {
        put(alt, y);
        T* p = cur;
        cur = alt;
        alt = p;
        __syncthreads();
      }
    }
  }
};

// rsum, csum: as launch_brick_down.  hy and oy are even, so row pairs are a
// lane's own.
template <typename T, bool PER, int LEN, int SEG, bool ZERO>
__global__ __launch_bounds__(64 * SEG) void k_win2_down(W2Args<T> A, const T* __restrict__ u0,
                                                        const T* __restrict__ b, T* __restrict__ u,
                                                        T* __restrict__ bc, double* __restrict__ rsum,
                                                        double* __restrict__ csum, Batch bt,
                                                        const int* __restrict__ stop) {
  __shared__ T E[2][SEG * 128];
  __shared__ double red[2][SEG];
  {
    const long long mb = blockIdx.y;
    if (!ZERO) u0 += mb * bt.s0;
    if (rsum != nullptr) rsum += mb * bt.part_stride;
    if (csum != nullptr) csum += mb * bt.part_stride;
    b += mb * bt.s0;
    u += mb * bt.s0;
    bc += mb * bt.s1;
    if (stop != nullptr) stop += mb * bt.stop_stride;
  }
  lds_poison(&E[0][0], 2 * SEG * 128);
  lds_poison(&red[0][0], 2 * SEG);
  lds_poison_sync();
  const Win2<T, PER, LEN, SEG> B(A, xcd_tile(blockIdx.x, A.nblk));
  T bb[LEN], y[LEN], r[LEN];
  T *cur = E[0], *alt = E[1];
  if constexpr (!ZERO) B.load(A, u0, y);
  B.load(A, b, bb);
  if (stop != nullptr && *stop) return;
  double r2 = 0.0, cs = 0.0;
  if constexpr (ZERO) {
#pragma unroll
    for (int m = 0; m < LEN; ++m) y[m] = (T)0;
  } else {
    B.put(cur, y);
    __syncthreads();
  }
  B.template relax<ZERO, true, !ZERO>(A, cur, alt, y, bb, r2);
  B.lap(A, cur, y, r);
  const int cnx = A.nx >> 1;
  const bool co = B.xown(A) && !(B.gx & 1);
#pragma unroll
  for (int m = 0; m < LEN; m += 2) {
    const T p = (bb[m] - r[m]) + (bb[m + 1] - r[m + 1]);
    const T v = (p + wshift<DPP_WAVE_SHL1>(p)) * (T)0.25;
    if (B.yown(A, m) && co) {
      (bc + (size_t)((B.gy + m) >> 1) * cnx)[B.gx >> 1] = v;
      cs += (double)v;
    }
  }
  B.store(A, u, y);
  if (rsum != nullptr || csum != nullptr) {
    r2 = wave_sum_dpp(r2);
    cs = wave_sum_dpp(cs);
    if (B.i == 0) {
      red[0][B.seg()] = r2;
      red[1][B.seg()] = cs;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = 0.0, c = 0.0;
#pragma unroll
      for (int q = 0; q < SEG; ++q) {
        t += red[0][q];
        c += red[1][q];
      }
      if (rsum != nullptr) rsum[blockIdx.x] = t;
      if (csum != nullptr) csum[2 * (size_t)blockIdx.x + 1] = c;
    }
  }
}

template <typename T, bool PER, int LEN, int SEG>
__global__ __launch_bounds__(64 * SEG) void k_win2_up(W2Args<T> A, const T* __restrict__ u, const T* __restrict__ e,
                                                      const T* __restrict__ b, T* __restrict__ out, Batch bt,
                                                      const int* __restrict__ stop) {
  __shared__ T E[2][SEG * 128];
  {
    const long long mb = blockIdx.y;
    u += mb * bt.s0;
    b += mb * bt.s0;
    out += mb * bt.s0;
    e += mb * bt.s1;
    if (stop != nullptr) stop += mb * bt.stop_stride;
  }
  lds_poison(&E[0][0], 2 * SEG * 128);
  lds_poison_sync();
  const Win2<T, PER, LEN, SEG> B(A, xcd_tile(blockIdx.x, A.nblk));
  T bb[LEN], y[LEN];
  // The segment's rows lie between coarse rows (gy - 1) >> 1 .. (gy + LEN) >> 1
  // (gy is even); each is interpolated in x once, ghosts with their sign.
  constexpr int NE = LEN / 2 + 2;
  T ep[NE], en[NE];
  const int cnx = A.nx >> 1, cny = A.ny >> 1;
  T sx = (T)1;
  {
    int I = B.gx >> 1, J = I + ((B.gx & 1) ? 1 : -1);
    if (PER) {
      I = ((I % cnx) + cnx) % cnx;
      J = ((J % cnx) + cnx) % cnx;
    } else {
      if (J < 0 || J >= cnx) sx = (T)-1;
      I = min(max(I, 0), cnx - 1);
      J = min(max(J, 0), cnx - 1);
    }
    const int kb = (B.gy >> 1) - 1;
#pragma unroll
    for (int p = 0; p < NE; ++p) {
      int K = kb + p;
      if (PER) K = ((K % cny) + cny) % cny;
      else K = min(max(K, 0), cny - 1);
      ep[p] = (e + (size_t)K * cnx)[I];
      en[p] = (e + (size_t)K * cnx)[J];
    }
  }
  B.load(A, u, y);
  B.load(A, b, bb);
  if (stop != nullptr && *stop) return;
  {
    const int kb = (B.gy >> 1) - 1;
    T x[NE];
#pragma unroll
    for (int p = 0; p < NE; ++p) {
      const T sy = (!PER && (kb + p < 0 || kb + p >= cny)) ? (T)-1 : (T)1;
      x[p] = sy * fma_of((T)3, ep[p], sx * en[p]);
    }
#pragma unroll
    for (int m = 0; m < LEN; ++m) {
      const T lo = x[(m + 1) >> 1], hi = x[((m + 1) >> 1) + 1];
      y[m] += ((m & 1) ? fma_of((T)3, lo, hi) : fma_of((T)3, hi, lo)) * (T)(1.0 / 16.0);
    }
  }
  T *cur = E[0], *alt = E[1];
  B.put(cur, y);
  __syncthreads();
  double none = 0.0;
  B.template relax<false, false, false>(A, cur, alt, y, bb, none);
  B.store(A, out, y);
}

template <typename T>
static bool w2_args(W2Args<T>& A, const LevelView<T>& L, int s, const StageCoef* co, int steps, int halo, int rows) {
  if (s < 1 || steps < 1 || s * steps > W2S || L.faces != nullptr || ((L.nx | L.ny) & 1)) return false;
  A.nx = L.nx;
  A.ny = L.ny;
  A.hx = A.hy = (halo + 1) & ~1;
  A.ox = 64 - 2 * A.hx;
  A.oy = rows - 2 * A.hy;
  A.tx = (L.nx + A.ox - 1) / A.ox;
  A.nblk = A.tx * ((L.ny + A.oy - 1) / A.oy);
  A.s = s;
  A.stages = s * steps;
  A.ihx = L.ihx2;
  A.ihy = L.ihy2;
  for (int q = 0; q < s; ++q) {
    A.co[q][0] = (T)co[q].mu;
    A.co[q][1] = (T)co[q].nu;
    A.co[q][2] = (T)co[q].c;
  }
  return true;
}

constexpr int W2SEG = 8;                // segments (wavefronts) of a window
constexpr int W2SMALL = 4, W2LARGE = 6;  // rows per segment
constexpr int W2SMALL_MAX = 1024;       // windows of short segments

// the smallest window: short segments, halo 6
size_t win2_blocks_max(int nx, int ny) {
  constexpr int oy = W2SMALL * W2SEG - 12;
  return (size_t)((nx + 51) / 52) * (size_t)((ny + oy - 1) / oy);
}

// Short segments while those windows are few (levels up to about 1024^2, where
// the serial work of a segment counts: a 256^2 float64 Dirichlet cycle 62.7 ->
// 58.7 us, 512^2 74.6 -> 70.4, 1024^2 103 -> 95), longer ones, with less halo,
// beyond (4096^2: 363 -> 355 us float64, 251 -> 233 float32).  Windows of 36, 60,
// 64, 72, 80, 96 and 128 rows were slower at either end.
template <typename T, typename F>
static int w2_launch(const LevelView<T>& L, int s, const StageCoef* co, int steps, int halo, F&& go) {
  W2Args<T> A;
  if (!w2_args(A, L, s, co, steps, halo, W2SMALL * W2SEG)) return 0;
  if (A.nblk <= W2SMALL_MAX) {
    go(A, std::integral_constant<int, W2SMALL>{});
  } else {
    w2_args(A, L, s, co, steps, halo, W2LARGE * W2SEG);
    go(A, std::integral_constant<int, W2LARGE>{});
  }
  return A.nblk;
}

template <typename T>
int launch_win2_down(const LevelView<T>& L, const T* u0, const T* b, T* u, T* bc, int s, const StageCoef* co,
                     int steps, double* rsum, double* csum, const int* stop, hipStream_t st, const Batch& bt) {
  const bool zero = u0 == nullptr;
  return w2_launch<T>(L, s, co, steps, s * steps + (zero ? 0 : 1), [&](const W2Args<T>& A, auto len) {
    constexpr int N = decltype(len)::value, G = W2SEG;
    auto k = L.periodic ? (zero ? k_win2_down<T, true, N, G, true> : k_win2_down<T, true, N, G, false>)
                        : (zero ? k_win2_down<T, false, N, G, true> : k_win2_down<T, false, N, G, false>);
    hipLaunchKernelGGL(k, dim3(A.nblk, bt.nb), dim3(64 * G), 0, st, A, u0, b, u, bc, rsum, csum, bt, stop);
  });
}

template <typename T>
int launch_win2_up(const LevelView<T>& L, const T* u, const T* e, const T* b, T* out, int s, const StageCoef* co,
                   int steps, const int* stop, hipStream_t st, const Batch& bt) {
  return w2_launch<T>(L, s, co, steps, s * steps, [&](const W2Args<T>& A, auto len) {
    constexpr int N = decltype(len)::value, G = W2SEG;
    auto k = L.periodic ? k_win2_up<T, true, N, G> : k_win2_up<T, false, N, G>;
    hipLaunchKernelGGL(k, dim3(A.nblk, bt.nb), dim3(64 * G), 0, st, A, u, e, b, out, bt, stop);
  });
}

#define RKL_WIN2_INST(T)                                                                                         \
  template int launch_win2_down<T>(const LevelView<T>&, const T*, const T*, T*, T*, int, const StageCoef*, int,  \
                                   double*, double*, const int*, hipStream_t, const Batch&);                     \
  template int launch_win2_up<T>(const LevelView<T>&, const T*, const T*, const T*, T*, int, const StageCoef*,   \
                                 int, const int*, hipStream_t, const Batch&);
RKL_WIN2_INST(double)
RKL_WIN2_INST(float)

}  // namespace rkl
