// Coarse tail of the V-cycle in one workgroup, column form.
//
// The same cycle as k_tail (tail.hip): from the first level of at most
// TAIL_MAX_CELLS cells down to the coarsest one and back, every array in LDS
// (Sec. 2.1; stage recurrence of App. A, ghosts of Sec. 2.3), for RKL smoothing
// of up to four stages and the direct coarsest solve (direct.h).
//
// One CU holds the whole level, so a stage is a chain of LDS latencies and
// barriers, not a matter of bandwidth: a 16^3 float64 stage moves 180 KB of LDS
// (about 1400 cycles) and took 3500 in k_tail.  1024 threads each own up to TCM
// consecutive cells of one z column in registers.  Their z neighbours are the
// thread's own, a stage reads only the x and y neighbours and the column's two
// ends from LDS, and writes each cell once (5.5 accesses a cell against 10 of
// the cell-by-cell sweep).  The number of cells per thread is a template
// parameter, picked per level by a uniform branch, so that a stage has no
// branch at all and its loads are in flight together (the same loops with a
// run-time count took 2700 - 4000 cycles a stage whatever the level's size;
// now 1000 - 2500).  Right-hand sides, iterates and residuals of a phase stay
// in registers and residuals reach the restriction already summed over pairs
// along the march.  A two-dimensional level marches its y axis (planes of one
// row).  A coarsest level of at most 64 cells is one product with its dense
// inverse (1100 cycles against 4800 of six axis products).
//
// Measured, k_tail -> this kernel: 16^3 .. 4^3 float64 33.0 -> 16.0 us
// (Dirichlet), 40.6 -> 17.7 (periodic); 12^3 .. float32 periodic 21.6 -> 12.6;
// 64^2 .. 4^2 float64 periodic 50.7 -> 18.6 us.
#include <algorithm>
#include <cstring>

#include "check.h"
#include "direct.h"

namespace rkl {

constexpr int TCNT = 1024;   // threads
constexpr int TCM = 4;       // most cells per thread
constexpr int TCS = 4;       // most stages per tau-step
constexpr int TCTAB = 1536;  // doubles of the direct solve's tables cached in LDS

template <typename T>
struct ColLevel {
  int nx, ny, nz, nxy, n;  // marching view: a 2-D level is nx x 1 x (its y)
  int len, seg, off;       // cells per segment, segments; first of the level's three LDS arrays
  int ragged;              // the last segment is shorter
  unsigned rxy, rx;        // 2^32 / nxy and 2^32 / nx, rounded up (exact quotients for indices below 2^16)
  T ihx, ihy, ihz;
  T co[TCS][3];            // stage coefficients mu, nu, c (mu_1 = 1, nu_1 = 0)
};

template <typename T>
struct ColArgs {
  int nlev, s, n_pre, n_post, doff, ntab;
  int dx, dy, dz;       // coarsest level as the direct solve sees it
  const double* dtab;   // its tables
  const double* dense;  // its 64 x 64 inverse (levels of at most 64 cells) or nullptr
  ColLevel<T> lv[TAIL_MAX_LEVELS];
};

// The thread's cells of a level: cell m is at element a + m nxy, m < cnt.
struct Col {
  int a, k0, cnt;
  int i, j;
};

template <typename T>
__device__ __forceinline__ Col col_of(const ColLevel<T>& V) {
  Col C;
  const int sg = (int)__umulhi(threadIdx.x, V.rxy);
  int q = (int)threadIdx.x - sg * V.nxy;
  C.k0 = sg * V.len;
  C.cnt = V.ragged ? min(V.nz - C.k0, V.len) : V.len;
  if (sg >= V.seg) q = C.k0 = C.cnt = 0;  // idle thread
  C.j = (int)__umulhi((unsigned)q, V.rx);
  C.i = q - C.j * V.nx;
  C.a = C.k0 * V.nxy + q;
  return C;
}

// Relaxation of one level by the workgroup.  LEN cells per thread, RAG: some
// threads own fewer.
template <typename T, bool PER, bool FLAT, int LEN, bool RAG>
struct ColWork {
  const Col& C;
  const T* co;    // LDS: the level's stage coefficients
  int nxy, last;
  int oxm, oxp, oym, oyp, ozl, ozh;  // neighbour offsets (0: the cell itself, a Dirichlet ghost)
  bool gxm, gxp, gym, gyp, gzl, gzh;
  T ihx, ihy, ihz;

  __device__ __forceinline__ ColWork(const ColLevel<T>& V, const Col& c, const T* coef) : C(c), co(coef) {
    nxy = V.nxy;
    last = RAG ? max(C.cnt - 1, 0) : LEN - 1;
    const int ke = C.k0 + last;
    gxm = !PER && C.i == 0;
    gxp = !PER && C.i == V.nx - 1;
    gym = !PER && C.j == 0;
    gyp = !PER && C.j == V.ny - 1;
    gzl = !PER && C.k0 == 0;
    gzh = !PER && ke == V.nz - 1;
    oxm = C.i > 0 ? -1 : (PER ? V.nx - 1 : 0);
    oxp = C.i < V.nx - 1 ? 1 : (PER ? 1 - V.nx : 0);
    oym = C.j > 0 ? -V.nx : (PER ? nxy - V.nx : 0);
    oyp = C.j < V.ny - 1 ? V.nx : (PER ? V.nx - nxy : 0);
    ozl = C.k0 > 0 ? -nxy : (PER ? V.n - nxy : 0);
    ozh = (ke < V.nz - 1 ? last + 1 : (PER ? last + 1 - V.nz : last)) * nxy;
    ihx = V.ihx;
    ihy = V.ihy;
    ihz = V.ihz;
  }

  // element of cell m next to the thread's first one (a missing cell reads the
  // last one's)
  __device__ __forceinline__ int at(int m) const { return (RAG ? min(m, last) : m) * nxy; }
  __device__ __forceinline__ void get(const T* Y, T (&v)[LEN]) const {
#pragma unroll
    for (int m = 0; m < LEN; ++m) v[m] = Y[C.a + at(m)];
  }
  __device__ __forceinline__ void put(T* Y, const T (&v)[LEN]) const {
    if (!RAG) {
      if (C.cnt > 0) {
#pragma unroll
        for (int m = 0; m < LEN; ++m) Y[C.a + m * nxy] = v[m];
      }
    } else {
#pragma unroll
      for (int m = 0; m < LEN; ++m)
        if (m < C.cnt) Y[C.a + m * nxy] = v[m];
    }
  }
  // M y at the thread's cells: Y holds the level, y the thread's own cells of
  // it; every load is unconditional, so all are in flight together
  __device__ __forceinline__ void lap(const T* Y, const T (&y)[LEN], T (&out)[LEN]) const {
    T xm[LEN], xp[LEN], ym[LEN], yp[LEN];
    const T* P = Y + C.a;
#pragma unroll
    for (int m = 0; m < LEN; ++m) {
      xm[m] = P[at(m) + oxm];
      xp[m] = P[at(m) + oxp];
      if (!FLAT) {
        ym[m] = P[at(m) + oym];
        yp[m] = P[at(m) + oyp];
      }
    }
    T zl = P[ozl], zh = P[ozh];
#pragma unroll
    for (int m = 0; m < LEN; ++m) {
      const T c = y[m];
      if (!PER) {
        if (gxm) xm[m] = -c;
        if (gxp) xp[m] = -c;
        if (!FLAT) {
          if (gym) ym[m] = -c;
          if (gyp) yp[m] = -c;
        }
      }
      T zm = m > 0 ? y[m > 0 ? m - 1 : 0] : zl;
      if (!PER && m == 0 && gzl) zm = -c;
      T zp;
      if (RAG) {
        const T up = y[m + 1 < LEN ? m + 1 : m];
        zp = m == last ? zh : up;
        if (!PER && m == last && gzh) zp = -c;
      } else {
        zp = m + 1 < LEN ? y[m + 1 < LEN ? m + 1 : m] : zh;
        if (!PER && m + 1 == LEN && gzh) zp = -c;
      }
      T v = ((xm[m] + xp[m]) - (T)2 * c) * ihx;
      if (!FLAT) v += ((ym[m] + yp[m]) - (T)2 * c) * ihy;
      out[m] = v + ((zm + zp) - (T)2 * c) * ihz;
    }
  }
  // `steps` tau-steps of s stages from y, which `cur` holds too unless `zero`
  // (the zero iterate, whose first stage is pointwise).  Stages alternate
  // between the level's two arrays; on return y is the result, and so is
  // `cur` after a barrier when `store`.
  __device__ __forceinline__ void relax(T*& cur, T*& alt, T (&y)[LEN], const T (&b)[LEN], int s, int steps, bool zero,
                                        bool store) const {
    T y2[LEN];
    int j = 0;
    const int total = steps * s;
    for (int t = 0; t < total; ++t) {
      const T mu = co[3 * j], nu = co[3 * j + 1], c = co[3 * j + 2];
      T w[LEN];
      if (zero && t == 0) {
#pragma unroll
        for (int m = 0; m < LEN; ++m) w[m] = (T)0;
      } else {
        lap(cur, y, w);
      }
#pragma unroll
      for (int m = 0; m < LEN; ++m) {
        const T old = y[m];
        const T before = j == 0 ? old : y2[m];  // stage 1: nu = 0
        y[m] = mu * old + nu * before + c * (w[m] - b[m]);
        y2[m] = old;
      }
      j = j + 1 == s ? 0 : j + 1;
      if (store || t + 1 < total) {
        put(alt, y);
        T* q = cur;
        cur = alt;
        alt = q;
        __syncthreads();
      }
    }
  }
};

// average of the children of a level-(l+1) cell (I, J, K) from the fine
// residual R in LDS: stored per cell, or summed over pairs along the march
template <typename T, bool FLAT>
__device__ __forceinline__ T col_children(const ColLevel<T>& F, const T* R, int I, int J, int K, bool zpair) {
  const int row = FLAT ? 0 : 2 * J * F.nx;
  const T* P = R + (zpair ? K : 2 * K) * F.nxy + row + 2 * I;
  T acc = P[0] + P[1];
  if (!FLAT) acc += P[F.nx] + P[F.nx + 1];
  if (!zpair) {
    const T* P1 = P + F.nxy;
    T up = P1[0] + P1[1];
    if (!FLAT) up += P1[F.nx] + P1[F.nx + 1];
    acc += up;
  }
  return acc * (FLAT ? (T)0.25 : (T)0.125);
}

// Pre-smoothing of a level from the zero iterate and its residual: b the
// thread's cells of the right-hand side (kept in LDS for the upstroke).  The
// residual is left in the array returned, summed over pairs along the march
// where LEN is even; `moved`: the iterate ended in the level's second array.
template <typename T, bool PER, bool FLAT, int LEN, bool RAG>
__device__ __forceinline__ T* col_down(const ColLevel<T>& V, const Col& C, const T* co, T* base, const T (&b4)[TCM],
                                       int s, int n_pre, bool& moved) {
  const ColWork<T, PER, FLAT, LEN, RAG> W(V, C, co);
  T *cur = base, *alt = base + V.n;
  T b[LEN], y[LEN], r[LEN];
#pragma unroll
  for (int m = 0; m < LEN; ++m) {
    b[m] = b4[m];
    y[m] = (T)0;
  }
  W.put(base + 2 * V.n, b);
  W.relax(cur, alt, y, b, s, n_pre, true, true);
  moved = cur != base;
  W.lap(cur, y, r);
#pragma unroll
  for (int m = 0; m < LEN; ++m) r[m] = b[m] - r[m];
  if constexpr (LEN % 2 == 0 && !RAG) {
    T* P = alt + ((C.k0 >> 1) * V.nxy + (C.a - C.k0 * V.nxy));
    if (C.cnt > 0) {
#pragma unroll
      for (int m = 0; m < LEN; m += 2) P[(m >> 1) * V.nxy] = r[m] + r[m + 1 < LEN ? m + 1 : m];
    }
  } else {
    W.put(alt, r);
  }
  __syncthreads();
  return alt;
}

// Prolongation + correction and post-smoothing of a level: E the coarser
// level's correction.  A coarse plane's x-y interpolation serves the fine cells
// around it in the thread's column: fine cell k lies between coarse planes
// (k - 1) >> 1 and the next one, weighing 3 and 1 (odd k) or 1 and 3.  The
// result is in `cur`, or leaves for u_top from registers.
template <typename T, bool PER, bool FLAT, int LEN, bool RAG>
__device__ __forceinline__ void col_up(const ColLevel<T>& V, const ColLevel<T>& N, const Col& C, const T* co,
                                       const T* E, T* base, bool moved, int s, int n_post, T* u_top, bool& now) {
  const ColWork<T, PER, FLAT, LEN, RAG> W(V, C, co);
  T* cur = moved ? base + V.n : base;
  T* alt = moved ? base : base + V.n;
  T y[LEN], b[LEN];
  W.get(cur, y);
  W.get(base + 2 * V.n, b);
  const int x0 = C.i >> 1;
  int x1 = x0 + ((C.i & 1) ? 1 : -1), y0 = 0, y1 = 0;
  T gx = (T)1, gy = (T)1;
  if (PER) x1 = x1 < 0 ? x1 + N.nx : (x1 >= N.nx ? x1 - N.nx : x1);
  else if (x1 < 0 || x1 >= N.nx) {
    x1 = x0;
    gx = (T)-1;
  }
  if (!FLAT) {
    y0 = C.j >> 1;
    y1 = y0 + ((C.j & 1) ? 1 : -1);
    if (PER) y1 = y1 < 0 ? y1 + N.ny : (y1 >= N.ny ? y1 - N.ny : y1);
    else if (y1 < 0 || y1 >= N.ny) {
      y1 = y0;
      gy = (T)-1;
    }
  }
  const int o00 = y0 * N.nx + x0, o01 = y0 * N.nx + x1, o10 = y1 * N.nx + x0, o11 = y1 * N.nx + x1;
  const int kb = (C.k0 - 1) >> 1;
  constexpr int NE = LEN / 2 + 2;  // planes (k0 - 1) >> 1 .. (k0 + LEN) >> 1
  T e[NE];
#pragma unroll
  for (int p = 0; p < NE; ++p) {
    int kp = kb + p;
    T gz = (T)1;
    if (PER) kp = kp < 0 ? kp + N.nz : (kp >= N.nz ? kp - N.nz : kp);
    else if (kp < 0) {
      kp = 0;
      gz = (T)-1;
    } else if (kp >= N.nz) {
      kp = N.nz - 1;
      gz = (T)-1;
    }
    kp = min(kp, N.nz - 1);  // (planes past what a short last segment uses)
    const T* P = E + kp * N.nxy;
    T v = (T)3 * P[o00] + gx * P[o01];
    if (!FLAT) v = (T)3 * v + gy * ((T)3 * P[o10] + gx * P[o11]);
    e[p] = gz * v;
  }
  const T pw = FLAT ? (T)(1.0 / 16.0) : (T)(1.0 / 64.0);
  const bool odd0 = C.k0 & 1;
#pragma unroll
  for (int m = 0; m < LEN; ++m) {
    constexpr bool EVEN = LEN % 2 == 0 && !RAG;  // every k0 is even
    const T ec = e[(m + 1) >> 1], ed = e[((m + 1) >> 1) + 1 < NE ? ((m + 1) >> 1) + 1 : NE - 1];
    if (EVEN) {
      y[m] += ((m & 1) ? (T)3 * ec + ed : ec + (T)3 * ed) * pw;
    } else {
      const T ea = e[m >> 1], eb = e[(m >> 1) + 1];
      const T lo = odd0 ? ea : ec, hi = odd0 ? eb : ed;
      const bool kodd = ((m & 1) != 0) != odd0;
      const T a3 = (T)3 * lo + hi, b3 = lo + (T)3 * hi;
      y[m] += (kodd ? a3 : b3) * pw;
    }
  }
  if (n_post > 0 || u_top == nullptr) {
    W.put(cur, y);
    __syncthreads();
    W.relax(cur, alt, y, b, s, n_post, false, u_top == nullptr);
  }
  now = cur != base;
  if (u_top != nullptr) W.put(u_top, y);
}

template <typename T, bool PER, bool FLAT>
__global__ __launch_bounds__(TCNT) void k_tail_col(ColArgs<T> A, const T* __restrict__ b_top, T* __restrict__ u_top,
                                                   Batch bt, const int* __restrict__ stop, CheckArgs chk) {
  extern __shared__ __align__(16) unsigned char pool_raw[];
  __shared__ double red[TCNT / WAVE];
  __shared__ double stab[TCTAB];
  __shared__ T sco[TAIL_MAX_LEVELS][TCS * 3];
  __shared__ int bad;
  {
    const long long mb = blockIdx.x;  // one workgroup per member
    b_top += mb * bt.s0;
    u_top += mb * bt.s0;
    if (stop != nullptr) stop += mb * bt.stop_stride;
    chk.part += mb * chk.part_stride;
    chk.res0sq += mb;
    chk.cs += mb;
    int cells = 0;  // the pool holds three arrays per level
    for (int l = 0; l < A.nlev; ++l) cells += 3 * A.lv[l].n;
    lds_poison(reinterpret_cast<T*>(pool_raw), cells);
    lds_poison(reinterpret_cast<double*>(pool_raw) + A.doff, 2 * A.lv[A.nlev - 1].n);
    lds_poison(red, TCNT / WAVE);
    lds_poison(stab, TCTAB);
    lds_poison(&sco[0][0], TAIL_MAX_LEVELS * TCS * 3);
    lds_poison_sync();
  }
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int nl = A.nlev;
  T* pool = reinterpret_cast<T*>(pool_raw);
  double* D0 = reinterpret_cast<double*>(pool_raw) + A.doff;
  // everything that comes from HBM, in flight together: the stop flag, the top
  // level's right-hand side, the direct solve's tables
  Col C = col_of<T>(A.lv[0]);
  T b[TCM];
  const int stopped = stop != nullptr ? *stop : 0;
  CheckLoads ck;
  if (chk.nblk > 0) check_load(chk, TCNT, ck);
#pragma unroll
  for (int m = 0; m < TCM; ++m) b[m] = m < C.cnt ? b_top[C.a + m * A.lv[0].nxy] : (T)0;
  double g[4];  // dense inverse: row tid / 16, columns 4 (tid % 16) ..
  if (A.dense != nullptr) {
#pragma unroll
    for (int m = 0; m < 4; ++m) g[m] = A.dense[4 * tid + m];
  }
  if (stopped) return;
  for (int q = tid; q < A.ntab; q += TCNT) stab[q] = A.dtab[q];
  if (tid < nl * TCS * 3) sco[tid / (TCS * 3)][tid % (TCS * 3)] = A.lv[tid / (TCS * 3)].co[(tid % (TCS * 3)) / 3][tid % 3];
  if (tid == 0) bad = 0;
  const double* tab = A.ntab > 0 ? stab : A.dtab;
  if (PER) {  // the right-hand side made mean-free
    double sm = 0.0;
#pragma unroll
    for (int m = 0; m < TCM; ++m) sm += (double)b[m];
    sm = wave_sum_dpp(sm);
    if (lane == 0) red[w] = sm;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < TCNT / WAVE; ++q) t += red[q];
    const T mean = (T)(t / (double)A.lv[0].n);
#pragma unroll
    for (int m = 0; m < TCM; ++m) b[m] -= mean;
  } else {
    __syncthreads();
  }
  unsigned swapped = 0u;  // bit l: the level's iterate is in its second array
  // downstroke: b holds the thread's cells of level l's right-hand side
  for (int l = 0; l < nl - 1; ++l) {
    const ColLevel<T>& V = A.lv[l];
    const ColLevel<T>& N = A.lv[l + 1];
    T* base = pool + V.off;
    bool moved = false;
    const T* R;
    bool zpair = false;
    if (V.ragged) {
      R = col_down<T, PER, FLAT, 4, true>(V, C, sco[l], base, b, A.s, A.n_pre, moved);
    } else if (V.len == 1) {
      R = col_down<T, PER, FLAT, 1, false>(V, C, sco[l], base, b, A.s, A.n_pre, moved);
    } else if (V.len == 2) {
      R = col_down<T, PER, FLAT, 2, false>(V, C, sco[l], base, b, A.s, A.n_pre, moved);
      zpair = true;
    } else if (V.len == 3) {
      R = col_down<T, PER, FLAT, 3, false>(V, C, sco[l], base, b, A.s, A.n_pre, moved);
    } else {
      R = col_down<T, PER, FLAT, 4, false>(V, C, sco[l], base, b, A.s, A.n_pre, moved);
      zpair = true;
    }
    if (moved) swapped |= 1u << l;
    // b_{l+1} = R(b_l - M u_l) at the thread's cells of the next level
    if (l + 1 < nl - 1) {
      C = col_of<T>(N);
#pragma unroll
      for (int m = 0; m < TCM; ++m)
        b[m] = m < C.cnt ? col_children<T, FLAT>(V, R, C.i, C.j, C.k0 + m, zpair) : (T)0;
    } else {
      for (int q = tid; q < N.n; q += TCNT) {
        const int K = (int)__umulhi((unsigned)q, N.rxy), p = q - K * N.nxy;
        const int J = (int)__umulhi((unsigned)p, N.rx);
        const double v = (double)col_children<T, FLAT>(V, R, p - J * N.nx, J, K, zpair);
        D0[q] = v;
        if (!(v * v <= 1.7976931348623157e308)) bad = 1;
      }
    }
  }
  // Coarsest level, solved directly into its first array.  A right-hand side
  // whose square overflows or is NaN gives u = 0, as the iteration's stop test
  // does.
  {
    const ColLevel<T>& V = A.lv[nl - 1];
    T* U = pool + V.off;
    __syncthreads();
    if (A.dense != nullptr) {
      // row tid / 16 of the inverse times b, four columns a thread, summed over
      // the 16 lanes of a row
      const int k = 4 * (tid & 15), r = tid >> 4;
      double v = 0.0;
#pragma unroll
      for (int m = 0; m < 4; ++m)
        if (k + m < V.n) v += g[m] * D0[k + m];
      v += dpp_mov_f64<0x111, 0xf>(v);  // row_shr:1, 2, 4, 8: lane 15 of each row of 16 holds its sum
      v += dpp_mov_f64<0x112, 0xf>(v);
      v += dpp_mov_f64<0x114, 0xf>(v);
      v += dpp_mov_f64<0x118, 0xf>(v);
      if ((tid & 15) == 15 && r < V.n) U[r] = bad ? (T)0 : (T)v;
    } else {
      double* D1 = D0 + V.n;
      const int nx = A.dx, ny = A.dy, nz = A.dz, nxy = nx * ny;
      const double* qx = tab;
      const double* qy = qx + nx * nx;
      const double* qz = qy + ny * ny;
      const double* lam = qz + nz * nz;
      constexpr int nw = TCNT / WAVE;
      auto keep = [](int, int, double v) { return v; };
      auto div = [&](int k, int q, double v) {
        const double l = lam[q % nx] + lam[nx + q / nx] + lam[nx + ny + k];
        return l != 0.0 ? v / l : 0.0;
      };
      axis_apply<false>(D0, D1, qx, nx, 1, ny * nz, w, nw, lane, keep);
      __syncthreads();
      axis_apply<false>(D1, D0, qy, ny, nx, nx * nz, w, nw, lane, keep);
      __syncthreads();
      axis_apply<false>(D0, D1, qz, nz, nxy, nxy, w, nw, lane, div);
      __syncthreads();
      axis_apply<true>(D1, D0, qz, nz, nxy, nxy, w, nw, lane, keep);
      __syncthreads();
      axis_apply<true>(D0, D1, qy, ny, nx, nx * nz, w, nw, lane, keep);
      __syncthreads();
      axis_apply<true>(D1, D0, qx, nx, 1, ny * nz, w, nw, lane, keep);
      __syncthreads();
      const bool zero = bad != 0;
      for (int q = tid; q < V.n; q += TCNT) U[q] = zero ? (T)0 : (T)D0[q];
    }
    __syncthreads();
  }
  for (int l = nl - 2; l >= 0; --l) {
    const ColLevel<T>& V = A.lv[l];
    const ColLevel<T>& N = A.lv[l + 1];
    const T* E = pool + N.off + (((swapped >> (l + 1)) & 1u) ? N.n : 0);
    T* base = pool + V.off;
    const bool moved = (swapped >> l) & 1u;
    T* top = l == 0 ? u_top : nullptr;
    bool now = moved;
    C = col_of<T>(V);
    if (V.ragged) col_up<T, PER, FLAT, 4, true>(V, N, C, sco[l], E, base, moved, A.s, A.n_post, top, now);
    else if (V.len == 1) col_up<T, PER, FLAT, 1, false>(V, N, C, sco[l], E, base, moved, A.s, A.n_post, top, now);
    else if (V.len == 2) col_up<T, PER, FLAT, 2, false>(V, N, C, sco[l], E, base, moved, A.s, A.n_post, top, now);
    else if (V.len == 3) col_up<T, PER, FLAT, 3, false>(V, N, C, sco[l], E, base, moved, A.s, A.n_post, top, now);
    else col_up<T, PER, FLAT, 4, false>(V, N, C, sco[l], E, base, moved, A.s, A.n_post, top, now);
    swapped = (swapped & ~(1u << l)) | ((now ? 1u : 0u) << l);
  }
  if (chk.nblk > 0) check_finish<TCNT>(chk, ck, stab);  // (stab: last read before the upstroke)
}

// cells per thread of a level: the fewest whose segments fit the workgroup and
// divide the march evenly, else the fewest that fit, with a short last segment
template <typename T>
static bool col_level(ColLevel<T>& V, int nx, int ny, int nz, int flat) {
  V.nx = nx;
  V.ny = flat ? 1 : ny;
  V.nz = flat ? ny : nz;
  V.nxy = V.nx * V.ny;
  V.n = V.nxy * V.nz;
  V.rxy = (unsigned)(((1ull << 32) + V.nxy - 1) / V.nxy);
  V.rx = (unsigned)(((1ull << 32) + V.nx - 1) / V.nx);
  if (V.nxy > TCNT) return false;
  const int fit = TCNT / V.nxy;
  for (int ragged = 0; ragged < 2; ++ragged) {
    for (int len = 1; len <= TCM; ++len) {
      const int seg = (V.nz + len - 1) / len;
      if (seg > fit || (!ragged && V.nz % len)) continue;
      V.len = len;
      V.seg = seg;
      V.ragged = ragged;
      return true;
    }
  }
  return false;
}

void tail_col_prepare() {
  static const bool ok = [] {
    const void* k[] = {(const void*)k_tail_col<double, true, false>, (const void*)k_tail_col<double, false, false>,
                       (const void*)k_tail_col<double, true, true>,  (const void*)k_tail_col<double, false, true>,
                       (const void*)k_tail_col<float, true, false>,  (const void*)k_tail_col<float, false, false>,
                       (const void*)k_tail_col<float, true, true>,   (const void*)k_tail_col<float, false, true>};
    for (const void* f : k)
      (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)TAIL_MAX_LDS);
    return true;
  }();
  (void)ok;
}

template <typename T>
bool launch_tail_col(const TailShape& ts, const StageCoef* const* smooth, int s, int n_pre, int n_post, int periodic,
                     const T* b_top, T* u_top, const int* stop, hipStream_t st, const Batch& bt,
                     const DirectTables& dir, const CheckArgs* chk) {
  if (ts.nlev < 2 || s > TCS || n_pre < 1) return false;
  ColArgs<T> A;
  std::memset(&A, 0, sizeof(A));
  const bool flat = ts.nz[0] == 1 && ts.ihz2[0] == 0.0;
  A.nlev = ts.nlev;
  A.s = s;
  A.n_pre = n_pre;
  A.n_post = n_post;
  A.dtab = dir.tab;
  A.dense = dir.dense;
  A.dx = dir.nx;
  A.dy = dir.ny;
  A.dz = dir.nz;
  const int nt = dir.nx * (dir.nx + 1) + dir.ny * (dir.ny + 1) + dir.nz * (dir.nz + 1);
  // long axes keep their tables in device memory, and the dense inverse needs none
  A.ntab = nt <= TCTAB && dir.dense == nullptr ? nt : 0;
  int off = 0;
  for (int l = 0; l < ts.nlev; ++l) {
    ColLevel<T>& V = A.lv[l];
    if (!col_level(V, ts.nx[l], ts.ny[l], ts.nz[l], flat) && l < ts.nlev - 1) return false;
    V.off = off;
    off += 3 * V.n;
    V.ihx = (T)ts.ihx2[l];
    V.ihy = flat ? (T)0 : (T)ts.ihy2[l];
    V.ihz = flat ? (T)ts.ihy2[l] : (T)ts.ihz2[l];
    for (int j = 0; j < s; ++j) {
      V.co[j][0] = (T)smooth[l][j].mu;
      V.co[j][1] = (T)smooth[l][j].nu;
      V.co[j][2] = (T)smooth[l][j].c;
    }
  }
  const size_t pool = ((size_t)off * sizeof(T) + 15) / 16 * 16;
  const size_t shm = pool + 2 * (size_t)A.lv[ts.nlev - 1].n * sizeof(double);
  if (shm > TAIL_MAX_LDS) return false;
  A.doff = (int)(pool / sizeof(double));
  tail_col_prepare();
  auto k = periodic ? (flat ? k_tail_col<T, true, true> : k_tail_col<T, true, false>)
                    : (flat ? k_tail_col<T, false, true> : k_tail_col<T, false, false>);
  hipLaunchKernelGGL(k, dim3(bt.nb), dim3(TCNT), shm, st, A, b_top, u_top, bt, stop,
                     chk != nullptr ? *chk : CheckArgs{});
  return true;
}

template bool launch_tail_col<double>(const TailShape&, const StageCoef* const*, int, int, int, int, const double*,
                                      double*, const int*, hipStream_t, const Batch&, const DirectTables&,
                                      const CheckArgs*);
template bool launch_tail_col<float>(const TailShape&, const StageCoef* const*, int, int, int, int, const float*,
                                     float*, const int*, hipStream_t, const Batch&, const DirectTables&,
                                     const CheckArgs*);

}  // namespace rkl
