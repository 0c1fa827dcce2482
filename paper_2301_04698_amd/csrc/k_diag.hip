// Diagnostics of the state: FP64 horizontal means per level (the mean
// profiles the paper reports for its stratocumulus case, Sec. 4.1), the
// domain integrals of rho0 theta_l and rho0 q_t (conserved by the scheme,
// Sec. 2.4), kinetic energy, central divergence and CFL number.
#include <algorithm>

#include "les_device.h"

namespace lesmi {

namespace {

// What a thread gathers over its cells; the level's density is applied to the
// sums.
struct DiagSums {
  double s[11];  // thl, qt, ql, u, v, w, w^2, w^3, b, u^2 + v^2 + w^2, div^2
  double dmax, cmax;
};
constexpr int kDiagParts = 13;  // values of a part of a level

// blockIdx.x: part of level blockIdx.y's rows.  A wave takes a row at a time,
// so that a cell's indices need no division; the sums run over a fixed order
// and are deterministic.  Bound by memory, 7 fields read once: 256 x 256 x 128
// FP32 63 us (74 with two barriers per value summed); with one block per level
// (128 of 256 CUs, a 64-bit division per cell) it took 289 us.
template <typename T>
__global__ __launch_bounds__(kBlock) void diag_kernel(Grid g, Profiles<T> P,
                                                      const T *__restrict__ u,
                                                      const T *__restrict__ v,
                                                      const T *__restrict__ w,
                                                      const T *__restrict__ thl,
                                                      const T *__restrict__ qt,
                                                      const T *__restrict__ ql,
                                                      const T *__restrict__ b,
                                                      double *__restrict__ parts) {
  const int k = blockIdx.y, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int kp = min(k + 1, g.nz - 1), km = max(k - 1, 0);
  // w changes sign across the walls
  const double sp = k + 1 < g.nz ? 1.0 : -1.0, sm = k > 0 ? 1.0 : -1.0;
  const double r0 = P.rho0[k], rm = P.rho0[km] * sm, rp = P.rho0[kp] * sp;
  const double hx = 0.5 / g.dx, hy = 0.5 / g.dy, hz = 0.5 / g.dz;
  const double cx = g.dt / g.dx, cy = g.dt / g.dy, cz = g.dt / g.dz;
  DiagSums a;
#pragma unroll
  for (int m = 0; m < 11; ++m) a.s[m] = 0.0;
  a.dmax = a.cmax = 0.0;
  constexpr int NW = kBlock / 64;
  const int64_t lev = g.nxy * k;
  for (int j = (int)blockIdx.x * NW + wave; j < g.ny; j += (int)gridDim.x * NW) {
    const int64_t row = lev + g.sy * j;
    const int64_t yp = lev + g.sy * pwrap(j + 1, g.ny), ym = lev + g.sy * pwrap(j - 1, g.ny);
    const int64_t zp = g.nxy * kp + g.sy * j, zm = g.nxy * km + g.sy * j;
    for (int i = lane; i < g.nx; i += 64) {
      const int64_t q = row + i;
      const int ip = pwrap(i + 1, g.nx), im = pwrap(i - 1, g.nx);
      const double uu = u[q], vv = v[q], ww = w[q];
      const double div = r0 * ((double)u[row + ip] - (double)u[row + im]) * hx +
                         r0 * ((double)v[yp + i] - (double)v[ym + i]) * hy +
                         (rp * (double)w[zp + i] - rm * (double)w[zm + i]) * hz;
      a.s[0] += (double)thl[q];
      a.s[1] += (double)qt[q];
      a.s[2] += (double)ql[q];
      a.s[3] += uu;
      a.s[4] += vv;
      a.s[5] += ww;
      a.s[6] += ww * ww;
      a.s[7] += ww * ww * ww;
      a.s[8] += (double)b[q];
      a.s[9] += uu * uu + vv * vv + ww * ww;
      a.s[10] += div * div;
      a.dmax = fmax(a.dmax, fabs(div));
      a.cmax = fmax(a.cmax, fabs(uu) * cx + fabs(vv) * cy + fabs(ww) * cz);
    }
  }
  // the waves' values, in order; one barrier for all of them
  __shared__ double red[NW][kDiagParts];
#pragma unroll
  for (int m = 0; m < 11; ++m) {
    const double s = wave_sum(a.s[m]);
    if (lane == 0) red[wave][m] = s;
  }
  const double dm = wave_max(a.dmax), cm = wave_max(a.cmax);
  if (lane == 0) {
    red[wave][11] = dm;
    red[wave][12] = cm;
  }
  __syncthreads();
  const int m = threadIdx.x;
  if (m >= kDiagParts) return;
  double s = red[0][m];
  for (int q = 1; q < NW; ++q) s = m < 11 ? s + red[q][m] : fmax(s, red[q][m]);
  parts[((int64_t)k * gridDim.x + blockIdx.x) * kDiagParts + m] = s;
}

// The parts of a level, in order, into its row of the output: thread m of
// block k the m-th value.
template <typename T>
__global__ __launch_bounds__(64) void diag_final_kernel(Profiles<T> P, int nparts,
                                                        const double *__restrict__ parts,
                                                        double *__restrict__ out) {
  const int k = blockIdx.x, m = threadIdx.x;
  if (m >= kDiagParts) return;
  const double *p = parts + (int64_t)k * nparts * kDiagParts + m;
  double s = p[0];
  for (int q = 1; q < nparts; ++q) {
    const double v = p[(int64_t)q * kDiagParts];
    s = m < 11 ? s + v : fmax(s, v);
  }
  const double r0 = P.rho0[k];
  double *o = out + (int64_t)k * kDiagStride;
  if (m < 9) o[m] = s;
  if (m < 2) o[9 + m] = r0 * s;
  if (m == 9) o[11] = 0.5 * r0 * s;
  if (m >= 10) o[m + 2] = s;
  if (m == 12) o[15] = 0.0;
}

}  // namespace

// Parts of a level: four blocks on each CU (eight: 4 us more at 256 x 256 x
// 128), rows for each of a block's waves.
static int diag_parts(const Grid &g) {
  const int rows = (g.ny + kBlock / 64 - 1) / (kBlock / 64);
  return std::max(1, std::min(rows, (1023 + g.nz) / g.nz));
}

size_t diag_part_values(const Grid &g) { return (size_t)g.nz * diag_parts(g) * kDiagParts; }

template <typename T>
void launch_diag(const Grid &g, const Profiles<T> &P, const T *u, const T *v, const T *w,
                 const T *thl, const T *qt, const T *ql, const T *b, double *parts,
                 double *level_sums, hipStream_t s) {
  const int n = diag_parts(g);
  diag_kernel<T><<<dim3(n, g.nz), kBlock, 0, s>>>(g, P, u, v, w, thl, qt, ql, b, parts);
  diag_final_kernel<T><<<g.nz, 64, 0, s>>>(P, n, parts, level_sums);
}

#define LES_INST(T)                                                                            \
  template void launch_diag<T>(const Grid &, const Profiles<T> &, const T *, const T *,        \
                               const T *, const T *, const T *, const T *, const T *, double *, \
                               double *, hipStream_t);
LES_INST(float)
LES_INST(double)
#undef LES_INST

}  // namespace lesmi
