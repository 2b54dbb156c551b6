// Direct coarsest solve of levels too large for one workgroup's LDS (the
// method is in direct.h).
//
// Three launches: every z plane is transformed in x and y by one workgroup
// (the plane and its x transform in LDS), every group of 16 (x, y) modes is
// transformed along z, divided by the eigenvalues and transformed back by one
// workgroup, and the planes are transformed back in y and x.  Planes beyond
// DIRECT_PLANE_LDS take one launch per axis instead, 16 lines a workgroup.
// The spectrum travels through one float64 array per member.  Bound by the
// latency of the three launches.  On the 50 x 30 x 22 coarsest level of a
// 200 x 120 x 88 Dirichlet box the accelerated RKL iteration it stands in for
// took about 530 stage launches and 30 host read-backs a cycle: the whole
// solve went from 33.2 to 1.84 ms.
#include "direct.h"
#include "host_common.h"

namespace rkl {

constexpr int DNT = 512;                               // threads per workgroup
constexpr size_t DIRECT_PLANE_LDS = 128 * 1024;        // LDS for a plane and its x transform
constexpr int DIRECT_MAX_AXIS = 512;                   // 2 x 16 lines of one axis in LDS: 128 KB

struct DirectArgs {
  int nx, ny, nz;
  const double *qx, *qy, *qz, *lx, *ly, *lz;  // eigenvector rows and eigenvalues (<= 0) of the axes
};

static DirectArgs direct_args(const DirectTables& D) {
  DirectArgs a{D.nx, D.ny, D.nz, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
  a.qx = D.tab;
  a.qy = a.qx + (size_t)D.nx * D.nx;
  a.qz = a.qy + (size_t)D.ny * D.ny;
  a.lx = a.qz + (size_t)D.nz * D.nz;
  a.ly = a.lx + D.nx;
  a.lz = a.ly + D.ny;
  return a;
}

// one z plane: FWD b -> spectrum in x and y, else spectrum -> u
template <typename T, bool FWD>
__global__ __launch_bounds__(DNT) void k_direct_plane(DirectArgs A, const T* __restrict__ b, double* __restrict__ W,
                                                      T* __restrict__ u, Batch bt, const int* __restrict__ stop) {
  extern __shared__ __align__(16) double dsm[];
  const int np = A.nx * A.ny;
  lds_poison(dsm, 2 * np);
  lds_poison_sync();
  {
    const long long mb = blockIdx.y;
    if (FWD) b += mb * bt.s0;
    else u += mb * bt.s0;
    W += mb * (long long)np * A.nz;
    if (stop != nullptr) stop += mb * bt.stop_stride;
  }
  if (stop != nullptr && *stop) return;
  const size_t p0 = (size_t)blockIdx.x * np;
  double* P = dsm;
  double* R = dsm + np;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  auto keep = [](int, int, double v) { return v; };
  for (int q = tid; q < np; q += DNT) P[q] = FWD ? (double)b[p0 + q] : W[p0 + q];
  __syncthreads();
  if (FWD) axis_apply<false>(P, R, A.qx, A.nx, 1, A.ny, w, DNT / WAVE, lane, keep);
  else axis_apply<true>(P, R, A.qy, A.ny, A.nx, A.nx, w, DNT / WAVE, lane, keep);
  __syncthreads();
  if (FWD) axis_apply<false>(R, P, A.qy, A.ny, A.nx, A.nx, w, DNT / WAVE, lane, keep);
  else axis_apply<true>(R, P, A.qx, A.nx, 1, A.ny, w, DNT / WAVE, lane, keep);
  __syncthreads();
  for (int q = tid; q < np; q += DNT) {
    if (FWD) W[p0 + q] = P[q];
    else u[p0 + q] = (T)P[q];
  }
}

// 16 lines of one axis (n cells, element stride s): MODE 0 forward, 1 inverse,
// 2 the z axis: forward, division by the eigenvalues, inverse
template <typename TI, typename TO, int MODE>
__global__ __launch_bounds__(DNT) void k_direct_axis(DirectArgs A, int axis, const TI* in, TO* out, long long sin,
                                                     long long sout, Batch bt, const int* __restrict__ stop) {
  extern __shared__ __align__(16) double dsm[];
  const int n = axis == 0 ? A.nx : (axis == 1 ? A.ny : A.nz);
  const int s = axis == 0 ? 1 : (axis == 1 ? A.nx : A.nx * A.ny);
  lds_poison(dsm, 32 * n);
  lds_poison_sync();
  {
    const long long mb = blockIdx.y;
    in += mb * sin;
    out += mb * sout;
    if (stop != nullptr) stop += mb * bt.stop_stride;
  }
  if (stop != nullptr && *stop) return;
  const double* Q = axis == 0 ? A.qx : (axis == 1 ? A.qy : A.qz);
  const int nlines = (int)((long long)A.nx * A.ny * A.nz / n);
  const int q0 = blockIdx.x * 16, nq = min(16, nlines - q0);
  double* P = dsm;           // [cell of the line][line]
  double* R = dsm + 16 * n;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  // neighbouring threads take neighbouring lines, except along x, where a
  // line's own cells are the contiguous ones
  auto at = [&](int e, int& c, int& l) -> size_t {
    if (axis == 0) {
      c = e % n;
      l = e / n;
    } else {
      l = e % nq;
      c = e / nq;
    }
    const int q = q0 + l;
    return (size_t)(q / s) * ((size_t)n * s) + q % s + (size_t)c * s;
  };
  for (int e = tid; e < n * nq; e += DNT) {
    int c, l;
    const size_t g = at(e, c, l);
    P[c * 16 + l] = (double)in[g];
  }
  __syncthreads();
  auto keep = [](int, int, double v) { return v; };
  // in LDS the 16 lines are an axis of stride 16
  if constexpr (MODE == 2) {
    axis_apply<false>(P, R, Q, n, 16, nq, w, DNT / WAVE, lane, [&](int k, int l, double v) {
      const int q = q0 + l;  // (x, y) mode: the line's place in a plane
      const double lam = A.lx[q % A.nx] + A.ly[q / A.nx] + A.lz[k];
      return lam != 0.0 ? v / lam : 0.0;
    });
    __syncthreads();
    axis_apply<true>(R, P, Q, n, 16, nq, w, DNT / WAVE, lane, keep);
    __syncthreads();
    R = P;
  } else {
    axis_apply<MODE == 1>(P, R, Q, n, 16, nq, w, DNT / WAVE, lane, keep);
    __syncthreads();
  }
  for (int e = tid; e < n * nq; e += DNT) {
    int c, l;
    const size_t g = at(e, c, l);
    out[g] = (TO)R[c * 16 + l];
  }
}

bool direct_axes_ok(int nx, int ny, int nz) {
  return nx <= DIRECT_MAX_AXIS && ny <= DIRECT_MAX_AXIS && nz <= DIRECT_MAX_AXIS;
}

// Raise the dynamic LDS limit of the kernels (once per process; a stream
// capture must not be the first caller).
void direct_prepare() {
  static const bool done = [] {
    const void* plane[] = {(const void*)k_direct_plane<double, true>, (const void*)k_direct_plane<double, false>,
                           (const void*)k_direct_plane<float, true>, (const void*)k_direct_plane<float, false>};
    for (const void* k : plane)
      (void)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)DIRECT_PLANE_LDS);
    const void* axis[] = {
        (const void*)k_direct_axis<double, double, 0>, (const void*)k_direct_axis<float, double, 0>,
        (const void*)k_direct_axis<double, double, 1>, (const void*)k_direct_axis<double, float, 1>,
        (const void*)k_direct_axis<double, double, 2>};
    for (const void* k : axis)
      (void)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)(32 * DIRECT_MAX_AXIS * sizeof(double)));
    return true;
  }();
  (void)done;
}

template <typename T>
void launch_direct(const DirectTables& D, const T* b, T* u, double* W, const int* stop, hipStream_t st,
                   const Batch& bt) {
  direct_prepare();
  const DirectArgs A = direct_args(D);
  const size_t np = (size_t)D.nx * D.ny, n = np * D.nz;
  const long long sw = (long long)n;
  auto lines = [&](int len) { return dim3((unsigned)((n / len + 15) / 16), bt.nb); };
  auto lds = [](int len) { return 32 * (size_t)len * sizeof(double); };
  const size_t pl = 2 * np * sizeof(double);
  const bool plane = pl <= DIRECT_PLANE_LDS;
  if (plane) {
    hipLaunchKernelGGL((k_direct_plane<T, true>), dim3(D.nz, bt.nb), dim3(DNT), pl, st, A, b, W, (T*)nullptr, bt, stop);
  } else {
    hipLaunchKernelGGL((k_direct_axis<T, double, 0>), lines(D.nx), dim3(DNT), lds(D.nx), st, A, 0, b, W, bt.s0, sw, bt,
                       stop);
    hipLaunchKernelGGL((k_direct_axis<double, double, 0>), lines(D.ny), dim3(DNT), lds(D.ny), st, A, 1, W, W, sw, sw,
                       bt, stop);
  }
  hipLaunchKernelGGL((k_direct_axis<double, double, 2>), lines(D.nz), dim3(DNT), lds(D.nz), st, A, 2, W, W, sw, sw, bt,
                     stop);
  if (plane) {
    hipLaunchKernelGGL((k_direct_plane<T, false>), dim3(D.nz, bt.nb), dim3(DNT), pl, st, A, (const T*)nullptr, W, u, bt,
                       stop);
  } else {
    hipLaunchKernelGGL((k_direct_axis<double, double, 1>), lines(D.ny), dim3(DNT), lds(D.ny), st, A, 1, W, W, sw, sw,
                       bt, stop);
    hipLaunchKernelGGL((k_direct_axis<double, T, 1>), lines(D.nx), dim3(DNT), lds(D.nx), st, A, 0, W, u, sw, bt.s0, bt,
                       stop);
  }
}

template void launch_direct<double>(const DirectTables&, const double*, double*, double*, const int*, hipStream_t,
                                    const Batch&);
template void launch_direct<float>(const DirectTables&, const float*, float*, double*, const int*, hipStream_t,
                                   const Batch&);

}  // namespace rkl
