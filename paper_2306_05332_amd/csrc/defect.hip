// Residual (defect) of a 3-D level: r = b - M u (Sec. 2.1 eq. residual, opposite
// sign), stored or only summed, with float64 partial sums of r^2 and r; and the
// same for u' = u + e (e float32), which it also writes: the mixed path's update
// of the float64 iterate folded into the next defect (Sec. 2.2.3), 32 bytes a
// cell against 20 + 20 for the update and the defect apart.  Ghosts as in Sec.
// 2.3, level-0 face data included.
//
// Bound by memory.  A wavefront takes 64 columns by DR rows and marches a few
// planes with its z neighbours in registers: x neighbours come from the adjacent
// lanes (the first and the last lane load theirs), y neighbours are the lane's own
// rows and one halo row on either side.  Workgroups are ordered chunk of planes
// by chunk of planes, and chunks are short, so the streams advance as compact
// fronts and a chunk's boundary planes are re-read from cache; within a chunk
// neighbouring rows stay on one XCD.
//
// Measured, float64 u and float32 r, 64 x 16 tiles in LDS (transfer.hip's form) ->
// here: 512^3 with the update 1027 -> 822 us (5.2 TB/s); 15 members of 96^3 108 ->
// 74, 16 of 64^3 30 -> 19, 128^3 17.7 -> 12.8, 11 of 32^3 10.7 -> 7.8.  (x
// neighbours of both end lanes in registers, 16 VGPRs more: 962 us at 512^3; the
// next planes loaded an iteration ahead, 20 more: 967.)
#include "host_common.h"
#include "kernels.h"

namespace rkl {

constexpr int DR = 4, DW = 4;  // rows per wavefront, wavefronts per workgroup

template <typename TU, typename TR, bool ADD, bool PER>
__global__ __launch_bounds__(WAVE * DW) void k_defect(LevelView<TU> F, const TU* __restrict__ u,
                                                      const TU* __restrict__ b, TR* __restrict__ out, int kz,
                                                      int gx, int per, double* __restrict__ part, Batch bt,
                                                      const int* __restrict__ stop, const float* __restrict__ e,
                                                      TU* __restrict__ unew) {
  __shared__ double red[2][DW];
  {
    const long long mb = blockIdx.y;
    if (u != nullptr) u += mb * bt.s0;
    if (ADD) {
      e += mb * bt.s0;
      unew += mb * bt.s0;
    }
    b += mb * bt.s0;
    if (out != nullptr) out += mb * bt.s0;
    part += mb * bt.part_stride;
    if (stop != nullptr) stop += mb * bt.stop_stride;
  }
  lds_poison(&red[0][0], 2 * DW);
  lds_poison_sync();
  if (stop != nullptr && *stop) return;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nx = F.nx, ny = F.ny, nz = F.nz;
  const size_t sxy = (size_t)nx * ny;
  const int chunk = blockIdx.x / per;
  const int tile = xcd_tile(blockIdx.x - chunk * per, per);
  // columns of the wavefront; the last tile of a row ends at the last column and
  // owns only what the tile before it does not
  const int x0 = (tile % gx) * WAVE, i = max(0, min(x0, nx - WAVE)) + lane;
  const int j0 = ((tile / gx) * DW + w) * DR;
  const int k0 = chunk * kz, k1 = min(k0 + kz, nz);
  const bool own = i >= x0 && i < nx;
  const int ic = min(i, nx - 1);
  // the first lane's left and the last lane's right neighbour (one lane is both
  // only where nx = 1, and both are then the cell itself)
  const bool last = lane == WAVE - 1 || i == nx - 1;
  const bool edge = lane == 0 || last;
  const int ie = lane == 0 ? (ic > 0 ? ic - 1 : (PER ? nx - 1 : 0)) : (ic < nx - 1 ? ic + 1 : (PER ? 0 : nx - 1));
  double s2 = 0.0, s1 = 0.0;
  if (j0 < ny) {
    size_t ro[DR + 2];  // row offsets of rows j0 - 1 .. j0 + DR, wrapped or clamped
#pragma unroll
    for (int r = 0; r < DR + 2; ++r) {
      const int j = j0 - 1 + r;
      const int q = PER ? ((j % ny) + ny) % ny : min(max(j, 0), ny - 1);
      ro[r] = (size_t)q * nx;
    }
    auto plane = [&](int k) -> size_t {
      const int q = PER ? (k < 0 ? k + nz : (k >= nz ? k - nz : k)) : min(max(k, 0), nz - 1);
      return (size_t)q * sxy;
    };
    auto val = [&](size_t row, int c) -> TU {
      if (u == nullptr) return (TU)0;
      TU v = (u + row)[c];
      if constexpr (ADD) v += (TU)(e + row)[c];
      return v;
    };
    TU zm[DR], c[DR + 2], ce[DR];  // planes k - 1 and k, and the end lanes' x neighbours
    auto load = [&](int k, TU(&v)[DR + 2], TU(&g)[DR]) {
      const size_t p = plane(k);
#pragma unroll
      for (int r = 0; r < DR + 2; ++r) v[r] = val(p + ro[r], ic);
#pragma unroll
      for (int r = 0; r < DR; ++r) g[r] = (TU)0;
      if (edge) {
#pragma unroll
        for (int r = 0; r < DR; ++r) g[r] = val(p + ro[r + 1], ie);
      }
    };
    {
      const size_t p = plane(k0 - 1);
#pragma unroll
      for (int r = 0; r < DR; ++r) zm[r] = val(p + ro[r + 1], ic);
    }
    load(k0, c, ce);
    for (int k = k0; k < k1; ++k) {
      TU n[DR + 2], ne[DR], bb[DR];
      const size_t p = (size_t)k * sxy;
#pragma unroll
      for (int r = 0; r < DR; ++r) bb[r] = (b + (p + ro[r + 1]))[ic];
      load(k + 1, n, ne);
#pragma unroll
      for (int r = 0; r < DR; ++r) {
        const int j = j0 + r;
        const TU v = c[r + 1];
        TU xm = wshift<DPP_WAVE_SHR1>(v), xp = wshift<DPP_WAVE_SHL1>(v);
        if (lane == 0) xm = ce[r];
        if (last) xp = ce[r];
        TU ym = c[r], yp = c[r + 2], zl = zm[r], zh = n[r + 1];
        if (!PER) {
          if (i == 0) xm = F.faces && j < ny ? dir_ghost(F, 0, (size_t)k * ny + j, v) : -v;
          if (i == nx - 1) xp = F.faces && j < ny ? dir_ghost(F, 1, (size_t)k * ny + j, v) : -v;
          if (j == 0) ym = dir_ghost(F, 2, (size_t)k * nx + ic, v);
          if (j == ny - 1) yp = dir_ghost(F, 3, (size_t)k * nx + ic, v);
          if (k == 0) zl = F.faces && j < ny ? dir_ghost(F, 4, (size_t)j * nx + ic, v) : -v;
          if (k == nz - 1) zh = F.faces && j < ny ? dir_ghost(F, 5, (size_t)j * nx + ic, v) : -v;
        }
        const TU res = bb[r] - lap7(v, xm, xp, ym, yp, zl, zh, F.ihx2, F.ihy2, F.ihz2);
        if (own && j < ny) {
          s2 += (double)res * (double)res;
          s1 += (double)res;
          const size_t o = p + ro[r + 1];
          if constexpr (ADD) {
            // non-temporal hints: the form runs on levels beyond the last-level
            // cache, where neither is read again before it would be evicted
            __builtin_nontemporal_store((TR)res, out + o + i);
            __builtin_nontemporal_store(v, unew + o + i);
          } else if (out != nullptr) {
            (out + o)[i] = (TR)res;
          }
        }
      }
#pragma unroll
      for (int r = 0; r < DR; ++r) {
        zm[r] = c[r + 1];
        ce[r] = ne[r];
      }
#pragma unroll
      for (int r = 0; r < DR + 2; ++r) c[r] = n[r];
    }
  }
  s2 = wave_sum_dpp(s2);
  s1 = wave_sum_dpp(s1);
  if (lane == 0) {
    red[0][w] = s2;
    red[1][w] = s1;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double a2 = 0.0, a1 = 0.0;
#pragma unroll
    for (int q = 0; q < DW; ++q) {
      a2 += red[0][q];
      a1 += red[1][q];
    }
    part[2 * (size_t)blockIdx.x] = a2;
    part[2 * (size_t)blockIdx.x + 1] = a1;
  }
}

struct DefectGrid {
  int gx, per, kz, nblk;
};

// Chunks of 16 planes, which keep what a chunk re-reads to an eighth and the
// streams' fronts compact (with the update, 512^3: 852 us in chunks of 8, 822 in
// 16; 15 members of 96^3 74 in either, 88 in 2), or of as many as still give
// about 1024 workgroups over all members.
static DefectGrid defect_grid(int nx, int ny, int nz, int nb) {
  DefectGrid g;
  g.gx = (nx + WAVE - 1) / WAVE;
  g.per = g.gx * ((ny + DR * DW - 1) / (DR * DW));
  g.kz = (int)std::max(1ll, std::min(16ll, (long long)g.per * nz * nb / 1024));
  g.nblk = g.per * ((nz + g.kz - 1) / g.kz);
  return g;
}

size_t defect_blocks(int nx, int ny, int nz, int nb) {
  if (nz == 1) return resid_blocks(nx, ny, nz);
  return (size_t)defect_grid(nx, ny, nz, nb).nblk;
}

template <typename TU, typename TR, bool ADD>
static void launch_defect(const LevelView<TU>& L, const TU* u, const TU* b, TR* r_out, double* part, const int* stop,
                          hipStream_t st, const Batch& bt, const float* e, TU* unew) {
  const DefectGrid g = defect_grid(L.nx, L.ny, L.nz, bt.nb);
  auto k = L.periodic ? k_defect<TU, TR, ADD, true> : k_defect<TU, TR, ADD, false>;
  hipLaunchKernelGGL(k, dim3(g.nblk, bt.nb), dim3(WAVE * DW), 0, st, L, u, b, r_out, g.kz, g.gx, g.per, part, bt,
                     stop, e, unew);
}

template <typename TU, typename TR>
void launch_defect_3d(const LevelView<TU>& L, const TU* u, const TU* b, TR* r_out, double* part, const int* stop,
                      hipStream_t st, const Batch& bt) {
  launch_defect<TU, TR, false>(L, u, b, r_out, part, stop, st, bt, nullptr, nullptr);
}

void launch_residual_add(const LevelView<double>& L, const double* u, const float* e, const double* b,
                         double* u_out, float* r_out, double* part, const int* stop, hipStream_t st) {
  if (L.nz == 1) fail(RKL_EINVAL, "the folded update is built for 3-D levels");
  if (u == nullptr || e == nullptr || u_out == nullptr || r_out == nullptr || u_out == u)
    fail(RKL_EINVAL, "folded update: bad buffers");
  launch_defect<double, float, true>(L, u, b, r_out, part, stop, st, single_batch(), e, u_out);
}

template void launch_defect_3d<double, double>(const LevelView<double>&, const double*, const double*, double*,
                                               double*, const int*, hipStream_t, const Batch&);
template void launch_defect_3d<double, float>(const LevelView<double>&, const double*, const double*, float*, double*,
                                              const int*, hipStream_t, const Batch&);
template void launch_defect_3d<float, float>(const LevelView<float>&, const float*, const float*, float*, double*,
                                             const int*, hipStream_t, const Batch&);

}  // namespace rkl
