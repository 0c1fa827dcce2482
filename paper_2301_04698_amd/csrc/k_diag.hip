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

// How a level is split.  A wave takes a unit at a time: a row, or where rows
// are fewer than waves one of the `pieces` of a row (`len` columns each), or
// where a row leaves more than half of the lanes idle the 64 / width rows that
// it holds side by side.
struct DiagSplit {
  int width;       // lanes of a row, a power of two: 64, or the least that hold a narrow row
  int pieces, len;
  int units, parts;  // of a level: units, blocks
};

// blockIdx.x: part of level blockIdx.y's units.  A cell's indices need no
// division; the sums run over a fixed order and are deterministic.  Bound by
// memory, 7 fields read once: 256 x 256 x 128 FP32 63 us (74 with two barriers
// per value summed); with one block per level (128 of 256 CUs, a 64-bit
// division per cell) it took 289 us.  With whole rows only, the call took 1795
// us at 51200 x 1 x 16 FP64 (359 with one block per level), 309 (180) at 5120 x
// 1 x 640, 81 (61) at 4 x 2048 x 64 FP32; with these units 62, 167 and 40.
template <typename T, bool NARROW>
__global__ __launch_bounds__(kBlock) void diag_kernel(Grid g, DiagSplit sp, Profiles<T> P,
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
  const double up = k + 1 < g.nz ? 1.0 : -1.0, dn = k > 0 ? 1.0 : -1.0;
  const double r0 = P.rho0[k], rm = P.rho0[km] * dn, rp = P.rho0[kp] * up;
  const double hx = 0.5 / g.dx, hy = 0.5 / g.dy, hz = 0.5 / g.dz;
  const double cx = g.dt / g.dx, cy = g.dt / g.dy, cz = g.dt / g.dz;
  DiagSums a;
#pragma unroll
  for (int m = 0; m < 11; ++m) a.s[m] = 0.0;
  a.dmax = a.cmax = 0.0;
  constexpr int NW = kBlock / 64;
  const int64_t lev = g.nxy * k;
  for (int n = (int)blockIdx.x * NW + wave; n < sp.units; n += (int)gridDim.x * NW) {
    int j, i0, i1;
    if (NARROW) {
      j = n * (64 / sp.width) + lane / sp.width;
      i0 = lane & (sp.width - 1);
      i1 = j < g.ny ? g.nx : 0;
      j = min(j, g.ny - 1);
    } else {
      j = n / sp.pieces;
      i0 = (n - j * sp.pieces) * sp.len;
      i1 = min(g.nx, i0 + sp.len);
      i0 += lane;
    }
    const int64_t row = lev + g.sy * j;
    const int64_t yp = lev + g.sy * pwrap(j + 1, g.ny), ym = lev + g.sy * pwrap(j - 1, g.ny);
    const int64_t zp = g.nxy * kp + g.sy * j, zm = g.nxy * km + g.sy * j;
    for (int i = i0; i < i1; i += 64) {
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

// Four blocks on each CU (eight: 4 us more at 256 x 256 x 128), and units for
// each of a block's waves.
static DiagSplit diag_split(const Grid &g) {
  constexpr int NW = kBlock / 64;
  const int most = (1023 + g.nz) / g.nz;
  DiagSplit d;
  d.width = 64;
  while (d.width >= 2 * g.nx) d.width /= 2;
  const int blocks = (g.nx + 63) / 64;  // of 64 columns
  const int want = std::min(blocks, std::max(1, most * NW / g.ny));
  d.len = (blocks + want - 1) / want * 64;
  d.pieces = (g.nx + d.len - 1) / d.len;
  const int rows = 64 / d.width;  // side by side
  d.units = (g.ny + rows - 1) / rows * d.pieces;
  d.parts = std::min((d.units + NW - 1) / NW, most);
  return d;
}

size_t diag_part_values(const Grid &g) { return (size_t)g.nz * diag_split(g).parts * kDiagParts; }

template <typename T>
void launch_diag(const Grid &g, const Profiles<T> &P, const T *u, const T *v, const T *w,
                 const T *thl, const T *qt, const T *ql, const T *b, double *parts,
                 double *level_sums, hipStream_t s) {
  const DiagSplit d = diag_split(g);
  const dim3 grid(d.parts, g.nz);
  if (d.width < 64)
    diag_kernel<T, true><<<grid, kBlock, 0, s>>>(g, d, P, u, v, w, thl, qt, ql, b, parts);
  else
    diag_kernel<T, false><<<grid, kBlock, 0, s>>>(g, d, P, u, v, w, thl, qt, ql, b, parts);
  diag_final_kernel<T><<<g.nz, 64, 0, s>>>(P, d.parts, parts, level_sums);
}

#define LES_INST(T)                                                                            \
  template void launch_diag<T>(const Grid &, const Profiles<T> &, const T *, const T *,        \
                               const T *, const T *, const T *, const T *, const T *, double *, \
                               double *, hipStream_t);
LES_INST(float)
LES_INST(double)
#undef LES_INST

}  // namespace lesmi
