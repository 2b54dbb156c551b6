// Small levels of the V-cycle, one launch per stroke.
//
// A level of 20^3 to 80^3 cells moves a few megabytes, all from cache: the strip
// kernels' marches there are chains of load latencies (a plane an iteration),
// and every launch adds its own start.  Here a workgroup takes a window of the
// level, halo included, in one burst of loads, runs every stage of the stroke on
// it in LDS and registers and writes the cells whose values are exact:
//   down  all n_pre tau-steps (Sec. 2.1 step 1; App. A), then the residual and
//         its restriction (steps 2a-2b, eq. restriction_example_3D): halo
//         n_pre s + 1, or n_pre s from the zero iterate (whose first stage is
//         pointwise),
//   up    prolongation and correction (steps 4-5, eq.
//         prolongation_example_3D), then the n_post tau-steps: halo n_post s.
// Values outside the exact region grow stale by one cell a stage and are never
// written.  Ghosts are those of Sec. 2.3: a window wraps round a periodic box and
// a Dirichlet face's ghost is minus the cell's own value.
//
// Window: 16 x 16 columns of four segments of LEN cells; a thread owns one
// segment.  x neighbours come from the adjacent lanes (a row of 16 is a DPP
// row), z neighbours are the thread's own cells, and only the y neighbours and
// the segment's two ends are read from LDS, all at once.  The arithmetic is the
// strip kernels', operation for operation, so either may run a level without a
// change of bits (a batch member's answer is the single solve's).
//
// Bound by the chain of one burst of loads, a barrier a stage and one store.
// Measured, separate passes -> here, float64: 32^3 down 14.2 -> 7.4 us, up 8.8 ->
// 7.6; 64^3 down 19.3 -> 9.8, up 12.3 -> 7.7.  32^3 Dirichlet solve 1091 -> 542 us
// together with the column tail, 256^3 periodic 5.26 -> 4.99 ms.
#include "host_common.h"
#include "kernels.h"

namespace rkl {

constexpr int BKX = 16, BKY = 16;      // window columns
constexpr int BKXY = BKX * BKY;
constexpr int BKSEG = 4;               // segments per column
constexpr int BKNT = BKXY * BKSEG;     // threads
constexpr int BKS = 4;                 // most stages per stroke

template <typename T>
struct BrickArgs {
  int nx, ny, nz;
  int tx, ty, nblk;   // tiles in x and y, all tiles
  int halo, ox, oy, oz;  // halo and exact cells of a window
  int s, stages;      // stages per tau-step and in all
  T ihx, ihy, ihz;
  T co[BKS][3];       // mu, nu, c of a tau-step's stages (mu_1 = 1, nu_1 = 0)
};

// value of the lane one to the left (SHR) or right within a row of 16 lanes
template <int CTRL>
__device__ __forceinline__ double row_shift(double v) {
  return dpp_mov_f64<CTRL, 0xf>(v);
}
template <int CTRL>
__device__ __forceinline__ float row_shift(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}

template <typename T, bool PER, int LEN>
struct Brick {
  static constexpr int NZ = BKSEG * LEN;
  int i, j, k0;     // the thread's column and first plane in the window
  int gx, gy, gz;   // and in the level (unwrapped)
  int a;            // LDS element of its first cell
  int oym, oyp, ozl, ozh;
  bool gxm, gxp, gym, gyp;
  unsigned in;      // bit m: cell m lies in the box (Dirichlet)
  int zlo, zhi;     // cells next to the z faces (Dirichlet; else -1)
  size_t col;       // element of the column in the level
  int z0;           // wrapped or unwrapped plane of cell 0

  __device__ __forceinline__ Brick(const BrickArgs<T>& A, int tile) {
    const int tid = threadIdx.x;
    i = tid & (BKX - 1);
    j = (tid / BKX) & (BKY - 1);
    k0 = (tid / BKXY) * LEN;
    const int bx = tile % A.tx, by = (tile / A.tx) % A.ty, bz = tile / (A.tx * A.ty);
    gx = bx * A.ox - A.halo + i;
    gy = by * A.oy - A.halo + j;
    gz = bz * A.oz - A.halo + k0;
    a = k0 * BKXY + j * BKX + i;
    oym = j > 0 ? -BKX : 0;
    oyp = j < BKY - 1 ? BKX : 0;
    ozl = k0 > 0 ? -BKXY : 0;
    ozh = (k0 + LEN < NZ ? LEN : LEN - 1) * BKXY;
    gxm = !PER && gx == 0;
    gxp = !PER && gx == A.nx - 1;
    gym = !PER && gy == 0;
    gyp = !PER && gy == A.ny - 1;
    zlo = PER ? -1 : -gz;
    zhi = PER ? -1 : A.nz - 1 - gz;
    in = 0u;
    int cx = gx, cy = gy;
    z0 = gz;
    if (PER) {
      cx = ((gx % A.nx) + A.nx) % A.nx;
      cy = ((gy % A.ny) + A.ny) % A.ny;
      z0 = ((gz % A.nz) + A.nz) % A.nz;
    } else if (gx >= 0 && gx < A.nx && gy >= 0 && gy < A.ny) {
#pragma unroll
      for (int m = 0; m < LEN; ++m)
        if (gz + m >= 0 && gz + m < A.nz) in |= 1u << m;
    }
    col = (size_t)cy * A.nx + cx;
  }
  // the thread's cells of a level array (0 outside a Dirichlet box)
  __device__ __forceinline__ void load(const BrickArgs<T>& A, const T* __restrict__ g, T (&v)[LEN]) const {
    const size_t sxy = (size_t)A.nx * A.ny;
    int z = z0;
#pragma unroll
    for (int m = 0; m < LEN; ++m) {
      v[m] = (T)0;
      if (PER || ((in >> m) & 1u)) v[m] = g[(size_t)z * sxy + col];
      ++z;
      if (PER && z == A.nz) z = 0;
    }
  }
  // cell m is one of the window's exact cells, in the box
  __device__ __forceinline__ bool own(const BrickArgs<T>& A, int m) const {
    return i >= A.halo && i < A.halo + A.ox && gx < A.nx && j >= A.halo && j < A.halo + A.oy && gy < A.ny &&
           k0 + m >= A.halo && k0 + m < A.halo + A.oz && gz + m < A.nz;
  }
  __device__ __forceinline__ void store(const BrickArgs<T>& A, T* __restrict__ g, const T (&v)[LEN]) const {
    const size_t sxy = (size_t)A.nx * A.ny;
#pragma unroll
    for (int m = 0; m < LEN; ++m)  // exact cells are never wrapped
      if (own(A, m)) g[(size_t)(gz + m) * sxy + (size_t)gy * A.nx + gx] = v[m];
  }
  __device__ __forceinline__ void put(T* Y, const T (&v)[LEN]) const {
#pragma unroll
    for (int m = 0; m < LEN; ++m) Y[a + m * BKXY] = v[m];
  }
  // M y at the thread's cells: Y holds the window, y the thread's own cells
  __device__ __forceinline__ void lap(const BrickArgs<T>& A, const T* Y, const T (&y)[LEN], T (&out)[LEN]) const {
    T ym[LEN], yp[LEN];
    const T* P = Y + a;
#pragma unroll
    for (int m = 0; m < LEN; ++m) {
      ym[m] = P[m * BKXY + oym];
      yp[m] = P[m * BKXY + oyp];
    }
    const T zl = P[ozl], zh = P[ozh];
#pragma unroll
    for (int m = 0; m < LEN; ++m) {
      const T c = y[m];
      T xm = row_shift<0x111>(c), xp = row_shift<0x101>(c);
      T zm = m > 0 ? y[m > 0 ? m - 1 : 0] : zl;
      T zp = m + 1 < LEN ? y[m + 1 < LEN ? m + 1 : m] : zh;
      if (!PER) {
        if (gxm) xm = -c;
        if (gxp) xp = -c;
        if (gym) ym[m] = -c;
        if (gyp) yp[m] = -c;
        if (m == zlo) zm = -c;
        if (m == zhi) zp = -c;
      }
      out[m] = lap7(c, xm, xp, ym[m], yp[m], zm, zp, A.ihx, A.ihy, A.ihz);
    }
  }
  // the stroke's stages from y, which `cur` holds too unless ZERO (the zero
  // iterate, whose first stage is pointwise); with LAST the result is left
  // in `cur` (after a barrier) as well as in y.  r2: sum of (M y - b)^2 of the
  // starting y over the thread's exact cells (not for ZERO).
  template <bool ZERO, bool LAST, bool SUM>
  __device__ __forceinline__ void relax(const BrickArgs<T>& A, T*& cur, T*& alt, T (&y)[LEN], const T (&b)[LEN],
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
#pragma unroll
        for (int m = 0; m < LEN; ++m) {
          const T res = w[m] - b[m];
          if (SUM && t == 0 && own(A, m)) r2 += (double)res * (double)res;
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

// rsum (optional, not ZERO): per workgroup, sum of (M u0 - b)^2 over its exact
// cells.  csum (optional): entry 2 blk + 1, sum of the coarse values it wrote.
template <typename T, bool PER, int LEN, bool ZERO>
__global__ __launch_bounds__(BKNT) void k_brick_down(BrickArgs<T> A, const T* __restrict__ u0,
                                                     const T* __restrict__ b, T* __restrict__ u, T* __restrict__ bc,
                                                     double* __restrict__ rsum, double* __restrict__ csum, Batch bt,
                                                     const int* __restrict__ stop) {
  __shared__ T Y[2][BKSEG * LEN * BKXY];
  __shared__ double red[BKNT / WAVE];
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
  lds_poison(&Y[0][0], 2 * BKSEG * LEN * BKXY);
  lds_poison(red, BKNT / WAVE);
  lds_poison_sync();
  const int tile = xcd_tile(blockIdx.x, A.nblk);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const Brick<T, PER, LEN> B(A, tile);
  T bb[LEN], y[LEN], r[LEN];
  T *cur = Y[0], *alt = Y[1];
  if constexpr (!ZERO) B.load(A, u0, y);
  B.load(A, b, bb);
  if (stop != nullptr && *stop) return;
  double r2 = 0.0;
  if constexpr (ZERO) {
#pragma unroll
    for (int m = 0; m < LEN; ++m) y[m] = (T)0;
  } else {
    B.put(cur, y);
    __syncthreads();
  }
  B.template relax<ZERO, true, !ZERO>(A, cur, alt, y, bb, r2);
  B.lap(A, cur, y, r);
#pragma unroll
  for (int m = 0; m < LEN; ++m) r[m] = bb[m] - r[m];
  B.put(alt, r);
  B.store(A, u, y);
  if constexpr (!ZERO) {
    r2 = wave_sum_dpp(r2);
    if (lane == 0) red[w] = r2;
  }
  __syncthreads();
  if constexpr (!ZERO) {
    if (rsum != nullptr && threadIdx.x == 0) {
      double t = 0.0;
#pragma unroll
      for (int q = 0; q < BKNT / WAVE; ++q) t += red[q];
      rsum[blockIdx.x] = t;
    }
  }
  double cs = 0.0;
  // coarse cells of the window: the 8-child average, summed as the strips do
  const int cx = A.ox >> 1, cy = A.oy >> 1, cz = A.oz >> 1;
  const int bx = tile % A.tx, by = (tile / A.tx) % A.ty, bz = tile / (A.tx * A.ty);
  const int gcx = A.nx >> 1, gcy = A.ny >> 1, gcz = A.nz >> 1;
  for (int q = threadIdx.x; q < cx * cy * cz; q += BKNT) {
    const int I = q % cx, J = (q / cx) % cy, K = q / (cx * cy);
    const int gi = bx * cx + I, gj = by * cy + J, gk = bz * cz + K;
    if (gi >= gcx || gj >= gcy || gk >= gcz) continue;
    const T* P = alt + (A.halo + 2 * K) * BKXY + (A.halo + 2 * J) * BKX + A.halo + 2 * I;
    const T z0 = (P[0] + P[BKX]) + (P[BKXY] + P[BKXY + BKX]);
    const T z1 = (P[1] + P[BKX + 1]) + (P[BKXY + 1] + P[BKXY + BKX + 1]);
    const T v = (z0 + z1) * (T)0.125;
    bc[((size_t)gk * gcy + gj) * gcx + gi] = v;
    cs += (double)v;
  }
  if (csum != nullptr) {
    __syncthreads();
    cs = wave_sum_dpp(cs);
    if (lane == 0) red[w] = cs;
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = 0.0;
#pragma unroll
      for (int q = 0; q < BKNT / WAVE; ++q) t += red[q];
      csum[2 * (size_t)blockIdx.x + 1] = t;
    }
  }
}

template <typename T, bool PER, int LEN>
__global__ __launch_bounds__(BKNT) void k_brick_up(BrickArgs<T> A, const T* __restrict__ u, const T* __restrict__ e,
                                                   const T* __restrict__ b, T* __restrict__ out, Batch bt,
                                                   const int* __restrict__ stop) {
  constexpr int CX = BKX / 2 + 2, CY = BKY / 2 + 2, CZ = BKSEG * LEN / 2 + 2;  // coarse window
  constexpr int CN = CX * CY * CZ, CPT = (CN + BKNT - 1) / BKNT;
  __shared__ T Y[2][BKSEG * LEN * BKXY];
  __shared__ T E[CN];
  {
    const long long mb = blockIdx.y;
    u += mb * bt.s0;
    b += mb * bt.s0;
    out += mb * bt.s0;
    e += mb * bt.s1;
    if (stop != nullptr) stop += mb * bt.stop_stride;
  }
  lds_poison(&Y[0][0], 2 * BKSEG * LEN * BKXY);
  lds_poison(E, CN);
  lds_poison_sync();
  const int tile = xcd_tile(blockIdx.x, A.nblk);
  const Brick<T, PER, LEN> B(A, tile);
  T bb[LEN], y[LEN];
  // the coarse window (one coarse cell around the fine one's parents), ghosts
  // with their sign
  {
    const int bx = tile % A.tx, by = (tile / A.tx) % A.ty, bz = tile / (A.tx * A.ty);
    const int hc = A.halo / 2 + 1;  // A.halo is even
    const int gcx = A.nx >> 1, gcy = A.ny >> 1, gcz = A.nz >> 1;
    auto cell = [](int q, int n, T& sg) {
      if (PER) return ((q % n) + n) % n;
      if (q < 0 || q >= n) sg = -sg;
      return min(max(q, 0), n - 1);
    };
    T ev[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      const int q = threadIdx.x + c * BKNT;
      ev[c] = (T)0;
      if (q < CN) {
        T sg = (T)1;
        const int I = cell(bx * (A.ox >> 1) - hc + q % CX, gcx, sg);
        const int J = cell(by * (A.oy >> 1) - hc + (q / CX) % CY, gcy, sg);
        const int K = cell(bz * (A.oz >> 1) - hc + q / (CX * CY), gcz, sg);
        ev[c] = sg * e[((size_t)K * gcy + J) * gcx + I];
      }
    }
    B.load(A, u, y);
    B.load(A, b, bb);
    if (stop != nullptr && *stop) return;
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      const int q = threadIdx.x + c * BKNT;
      if (q < CN) E[q] = ev[c];
    }
  }
  __syncthreads();
  // each coarse plane interpolated in x and y once for the column, then shared
  // by the fine planes around it: window plane k0 + m lies between coarse window
  // planes (k0 + m + 1) / 2 and the next
  {
    auto fma3 = [](T p, T q) -> T { return fma_of((T)3, p, q); };
    constexpr int NE = LEN / 2 + 2;
    const int ip = (B.i >> 1) + 1, in = ip + ((B.i & 1) ? 1 : -1);
    const int jp = (B.j >> 1) + 1, jn = jp + ((B.j & 1) ? 1 : -1);
    T x[NE];
#pragma unroll
    for (int p = 0; p < NE; ++p) {
      const T* R = E + ((B.k0 >> 1) + p) * (CX * CY);
      const T xp = fma3(R[jp * CX + ip], R[jp * CX + in]), xn = fma3(R[jn * CX + ip], R[jn * CX + in]);
      x[p] = fma3(xp, xn);
    }
#pragma unroll
    for (int m = 0; m < LEN; ++m) {
      const T lo = x[(m + 1) >> 1], hi = x[((m + 1) >> 1) + 1];
      y[m] += ((m & 1) ? fma3(lo, hi) : fma3(hi, lo)) * (T)(1.0 / 64.0);
    }
  }
  T *cur = Y[0], *alt = Y[1];
  B.put(cur, y);
  __syncthreads();
  double none = 0.0;
  B.template relax<false, false, false>(A, cur, alt, y, bb, none);
  B.store(A, out, y);
}

// Arguments and grid of a stroke of `steps` tau-steps with halo `halo`; false
// when the level does not take the window kernels.
template <typename T>
static bool brick_args(BrickArgs<T>& A, const LevelView<T>& L, int s, const StageCoef* co, int steps, int halo,
                       int len) {
  if (s < 1 || steps < 1 || s * steps > BKS || L.faces != nullptr || ((L.nx | L.ny | L.nz) & 1)) return false;
  A.nx = L.nx;
  A.ny = L.ny;
  A.nz = L.nz;
  A.halo = halo;
  A.ox = BKX - 2 * halo;
  A.oy = BKY - 2 * halo;
  A.oz = BKSEG * len - 2 * halo;
  A.tx = (L.nx + A.ox - 1) / A.ox;
  A.ty = (L.ny + A.oy - 1) / A.oy;
  A.nblk = A.tx * A.ty * ((L.nz + A.oz - 1) / A.oz);
  A.s = s;
  A.stages = s * steps;
  A.ihx = L.ihx2;
  A.ihy = L.ihy2;
  A.ihz = L.ihz2;
  for (int q = 0; q < s; ++q) {
    A.co[q][0] = (T)co[q].mu;
    A.co[q][1] = (T)co[q].nu;
    A.co[q][2] = (T)co[q].c;
  }
  return true;
}

// Segment length of a level's windows, 0 if the level stays with the strips: the
// shorter segments, else the longer ones (fewer windows), while every window (of
// all members) has a CU of its own; then likewise up to `most` windows.  A second
// window per CU still wins from the zero iterate and on the way up (72^3 below a
// 144^3 Dirichlet cycle: 181 -> 176 us float64, 152 -> 142 float32; up on level 0
// of a 96^3 cycle 111 -> 103), a third no longer (128^3 below 256^3: 450 -> 470),
// and with a given iterate, whose halo is wider, not even the second (64 x 32 x
// 64 solve 716 us on strips, 821 in 330 windows).
template <typename T>
static int brick_len(BrickArgs<T>& A, const LevelView<T>& L, int s, const StageCoef* co, int steps, int halo, int nb,
                     int most) {
  for (int limit = BRICK_SLOTS / 2; limit <= most; limit *= 2)
    for (int len : {4, 6}) {
      if (!brick_args(A, L, s, co, steps, halo, len)) return 0;
      if ((long long)A.nblk * nb <= limit) return len;
    }
  return 0;
}

template <typename T>
int launch_brick_down(const LevelView<T>& L, const T* u0, const T* b, T* u, T* bc, int s, const StageCoef* co,
                      int steps, double* rsum, double* csum, const int* stop, hipStream_t st, const Batch& bt) {
  if (fused_pinned<T>(L, s)) return 0;
  if (level_is_2d(L)) return launch_win2_down<T>(L, u0, b, u, bc, s, co, steps, rsum, csum, stop, st, bt);
  BrickArgs<T> A;
  const bool zero = u0 == nullptr;
  const int len = brick_len(A, L, s, co, steps, s * steps + (zero ? 0 : 1), bt.nb,
                            zero ? BRICK_SLOTS : BRICK_SLOTS / 2);
  if (len == 0) return 0;
  auto go = [&](auto k) {
    hipLaunchKernelGGL(k, dim3(A.nblk, bt.nb), dim3(BKNT), 0, st, A, u0, b, u, bc, rsum, csum, bt, stop);
    return A.nblk;
  };
  if (zero) {
    if (L.periodic) return len == 4 ? go(k_brick_down<T, true, 4, true>) : go(k_brick_down<T, true, 6, true>);
    return len == 4 ? go(k_brick_down<T, false, 4, true>) : go(k_brick_down<T, false, 6, true>);
  }
  if (L.periodic) return len == 4 ? go(k_brick_down<T, true, 4, false>) : go(k_brick_down<T, true, 6, false>);
  return len == 4 ? go(k_brick_down<T, false, 4, false>) : go(k_brick_down<T, false, 6, false>);
}

template <typename T>
bool launch_brick_up(const LevelView<T>& L, const T* u, const T* e, const T* b, T* out, int s, const StageCoef* co,
                     int steps, const int* stop, hipStream_t st, const Batch& bt) {
  if (fused_pinned<T>(L, s)) return false;
  if (level_is_2d(L)) return launch_win2_up<T>(L, u, e, b, out, s, co, steps, stop, st, bt) > 0;
  BrickArgs<T> A;
  const int len = brick_len(A, L, s, co, steps, (s * steps + 1) & ~1, bt.nb, BRICK_SLOTS);
  if (len == 0) return false;
  auto go = [&](auto k) {
    hipLaunchKernelGGL(k, dim3(A.nblk, bt.nb), dim3(BKNT), 0, st, A, u, e, b, out, bt, stop);
    return true;
  };
  if (L.periodic) return len == 4 ? go(k_brick_up<T, true, 4>) : go(k_brick_up<T, true, 6>);
  return len == 4 ? go(k_brick_up<T, false, 4>) : go(k_brick_up<T, false, 6>);
}

#define RKL_BRICK_INST(T)                                                                                          \
  template int launch_brick_down<T>(const LevelView<T>&, const T*, const T*, T*, T*, int, const StageCoef*, int,   \
                                    double*, double*, const int*, hipStream_t, const Batch&);                      \
  template bool launch_brick_up<T>(const LevelView<T>&, const T*, const T*, const T*, T*, int, const StageCoef*,   \
                                   int, const int*, hipStream_t, const Batch&);
RKL_BRICK_INST(double)
RKL_BRICK_INST(float)

}  // namespace rkl
